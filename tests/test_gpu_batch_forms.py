"""The launch forms of the batched decode (one, two or three launches): which
one a call takes, and the three-launch form's own branches, with max_packets
above 1024 so that short batches reach it.  Outputs are compared with the oracle
byte for byte; the form is read off the workspace, of which each form writes
different parts (the prefix sums in the two- and three-launch forms, the coarse
map in the two-launch form, the fine map in the three-launch form)."""
import numpy as np
import pytest

import oracle
import paper_1412_6862_amd as hm
from test_gpu_batch import _build_batch, _check_outputs, _expect, _to_dev

pytestmark = pytest.mark.gpu

FORMS = {(False, False, False): "one", (True, True, False): "two", (True, False, True): "three"}
MAX = 1100                       # above the packets of the one- and two-launch forms


def _poison(bd):
    bd.workspace.fill_(0xEE)


def _form(bd):
    """Form of the decode that ran since _poison (a batch of at least one tile)."""
    w = bd.workspace.cpu().numpy()
    a = 64 + 8 * (bd.max_packets + 1)
    b = a + 4 * (2 * bd.max_packets + 1024)
    return FORMS[tuple(bool((x[:4] != 0xEE).any()) for x in (w[64:a], w[a:b], w[b:]))]


def _decode(bd, own_stream=True, max_codewords=0):
    import torch

    bd.data.fill_(0x7777777777777777)
    bd.errpos.fill_(0x88)
    _poison(bd)
    s = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        bd.decode(stream=s, max_codewords=max_codewords)
    torch.cuda.synchronize()


@pytest.fixture
def config():
    """Sets the batch configuration and puts the old one back."""
    hm.hamming_batch_release_graphs()        # so that calls of this test get graphs of their own
    old, old_chunk = hm.hamming_batch_config_get(), hm.hamming_batch_chunk_get()

    def set_(schedule=3, grid_cap=0, use_graph=1, chunk_log2=3, xcd_chunk=1):
        hm.hamming_batch_config_set(schedule, xcd_chunk, grid_cap, use_graph)
        hm.hamming_batch_chunk_set(chunk_log2)

    yield set_
    hm.hamming_batch_config_set(*old)
    hm.hamming_batch_chunk_set(old_chunk)


MIB_WORDS = (1 << 20) // 8


@pytest.mark.parametrize("max_packets,mib,chunk_log2,grid_cap,form", [
    (256, 0, 0, 0, "one"), (257, 0, 0, 0, "two"), (1024, 0, 0, 0, "two"), (1025, 0, 0, 0, "three"),
    (256, 63, 0, 0, "one"), (256, 64, 0, 0, "two"), (256, 65, 3, 0, "one"), (256, 65, 0, 5, "two"),
    (1024, 255, 3, 0, "two"), (1024, 257, 0, 0, "three"), (1024, 257, 0, 5, "three"), (256, 300, 0, 5, "three")])
def test_batch_form_and_loads_either_side_of_their_bounds(gpu_device, config, max_packets, mib, chunk_log2, grid_cap,
                                                          form):
    """Short batches in arenas that put the call on either side of the bounds:
    packets and workgroups (before a grid cap) for the form, 64 MiB for the loads."""
    import torch

    arena, descs, ys = _build_batch(900 + max_packets, 60)
    cw = torch.zeros(max(arena.size, mib * MIB_WORDS), dtype=torch.int64, device=gpu_device)
    cw[:arena.size] = _to_dev(arena, gpu_device)
    bd = hm.BatchDecoder(cw, max_packets)
    bd.set_packets(descs)
    config(chunk_log2=chunk_log2)
    grid = hm.hamming_decode_batch_grid(cw.numel(), max_packets)
    config(chunk_log2=chunk_log2, grid_cap=grid_cap)
    assert form == ("one" if max_packets <= 256 and grid <= 4096 else
                    "two" if max_packets <= 1024 and grid <= 16384 else "three")
    _decode(bd)
    assert _form(bd) == form
    _check_outputs(bd, descs, _expect(ys, descs), data_fill=0x77, ep_fill=0x88)


@pytest.mark.parametrize("chunk_log2,fine_log2", [(0, 1), (0, 3), (0, 6), (2, 3), (3, 6), (1, 1)])
@pytest.mark.parametrize("schedule", [0, 1, 2, 3])
@pytest.mark.parametrize("use_graph", [0, 1])
def test_three_launches_grouped_fine_map(gpu_device, config, chunk_log2, fine_log2, schedule, use_graph):
    """A fine map of 2^fine_log2 tiles per entry, sized from the batch's tile
    count: where an entry spans several chunks every wave probes from it."""
    arena, descs, ys = _build_batch(1300 + fine_log2 + 7 * schedule + 50 * chunk_log2, 60)
    expect = _expect(ys, descs)
    config(schedule=schedule, use_graph=use_graph, chunk_log2=chunk_log2)
    cw = _to_dev(arena, gpu_device)
    full = hm.BatchDecoder(cw, MAX)
    full.set_packets(descs)
    _decode(full)
    tiles = full.totals()["tiles"]
    assert _form(full) == "three" and full.totals()["fine_log2"] == chunk_log2 and tiles >= 1 << fine_log2
    _check_outputs(full, descs, expect, data_fill=0x77, ep_fill=0x88)
    entries = (tiles >> fine_log2) + 1
    bd = hm.BatchDecoder(cw, MAX, workspace_bytes=hm.hamming_batch_workspace_min_bytes(MAX) - 4 + 4 * entries)
    bd.set_packets(descs)
    _decode(bd)
    assert _form(bd) == "three" and bd.totals()["fine_log2"] == fine_log2 and bd.totals()["tiles"] == tiles
    _check_outputs(bd, descs, expect, data_fill=0x77, ep_fill=0x88)


@pytest.mark.parametrize("schedule", [0, 1, 2, 3])
@pytest.mark.parametrize("grid_cap", [0, 3])
@pytest.mark.parametrize("one_entry", [0, 1])
def test_three_launches_many_tiny_and_empty_packets(gpu_device, config, schedule, grid_cap, one_entry):
    """1100 tiny and empty packets, with a whole fine map and with a single
    entry, from which every wave probes through runs of packets without tiles."""
    rng = np.random.default_rng(1400 + schedule)
    sizes = [int(rng.choice([0, 0, 1, 5, 64, 127, 128, 129, 300])) for _ in range(MAX)]
    rs = [int(rng.integers(3, 8)) for _ in range(MAX)]
    arena, descs, ys = _build_batch(1500 + schedule, MAX, sizes=sizes, rs=rs)
    config(schedule=schedule, grid_cap=grid_cap, chunk_log2=0)
    bd = hm.BatchDecoder(_to_dev(arena, gpu_device), MAX,
                         workspace_bytes=hm.hamming_batch_workspace_min_bytes(MAX) if one_entry else None)
    bd.set_packets(descs)
    _decode(bd)
    t = bd.totals()
    assert _form(bd) == "three" and t["tiles"] > 64 and t["packets"] == MAX
    assert ((t["tiles"] >> t["fine_log2"]) == 0) == bool(one_entry)
    assert not bd.status.cpu().numpy().any()
    _check_outputs(bd, descs, _expect(ys, descs), data_fill=0x77, ep_fill=0x88)


@pytest.mark.parametrize("n_packets", [1 << 19, (1 << 19) + 1, (1 << 19) + 257, (1 << 19) + 4099])
def test_three_launches_map_of_many_entries(gpu_device, config, n_packets):
    """A packet of one (63,57) codeword per fine-map entry, either side of the
    map size from which a wave fills 256 entries."""
    rng = np.random.default_rng(n_packets)
    cw = rng.integers(0, 1 << 63, n_packets, dtype=np.uint64)
    data, errpos = oracle.decode(cw, 6)
    bits = np.unpackbits(data.view(np.uint8), bitorder="little")[:n_packets * 57].reshape(n_packets, 57)
    want = np.packbits(np.pad(bits, ((0, 0), (0, 7))), axis=1, bitorder="little").view(np.uint64)[:, 0]
    descs = np.zeros(n_packets, dtype=hm.packet_dtype())
    descs["in_word_off"], descs["n_cw"], descs["r"] = np.arange(n_packets), 1, 6
    config(chunk_log2=0)
    bd = hm.BatchDecoder(_to_dev(cw, gpu_device), n_packets)
    bd.set_packets(descs)
    _decode(bd)
    t = bd.totals()
    assert t["tiles"] == n_packets and t["fine_log2"] == 0 and not bd.status.cpu().numpy().any()
    got = bd.data.cpu().numpy().view(np.uint64)[descs["data_word_off"].astype(np.int64)]
    assert np.array_equal(got, want)
    assert np.array_equal(bd.errpos.cpu().numpy()[descs["errpos_off"].astype(np.int64)], errpos)


@pytest.mark.parametrize("one_entry", [0, 1])
def test_three_launches_graph_serves_changing_counts(gpu_device, config, one_entry):
    """One graph, several packet counts read on the device (none among them),
    with eager work between the replays; then the same arguments without one."""
    import torch

    arena, descs, ys = _build_batch(1600 + one_entry, 30)
    expect = _expect(ys, descs)
    bd = hm.BatchDecoder(_to_dev(arena, gpu_device), MAX,
                         workspace_bytes=hm.hamming_batch_workspace_min_bytes(MAX) if one_entry else None)
    bd.set_packets(descs)
    s = torch.cuda.Stream()
    for use_graph, counts in ((1, (30, 7, 0, 19, 30, 1)), (0, (30, 0, 5))):
        config(use_graph=use_graph, chunk_log2=0)
        for n in counts:
            bd.data.fill_(0x3333333333333333)
            bd.errpos.fill_(0x44)
            bd.n_dev.fill_(n)
            _poison(bd)
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                bd.decode(stream=s)
            torch.cuda.synchronize()
            assert bd.totals()["packets"] == n
            if bd.totals()["tiles"]:
                assert _form(bd) == "three"
            _check_outputs(bd, descs[:n], expect[:n], data_fill=0x33, ep_fill=0x44)
