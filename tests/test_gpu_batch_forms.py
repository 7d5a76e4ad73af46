"""The launch forms of the batched decode (one, two or three launches): which
one a call takes.  Outputs are compared with the oracle
byte for byte; the form is read off the workspace, of which each form writes
different parts (the prefix sums in the two- and three-launch forms, the coarse
map in the two-launch form, the fine map in the three-launch form)."""
import pytest

import paper_1412_6862_amd as hm
from test_gpu_batch import _build_batch, _check_outputs, _expect, _to_dev

pytestmark = pytest.mark.gpu

FORMS = {(False, False, False): "one", (True, True, False): "two", (True, False, True): "three"}


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
