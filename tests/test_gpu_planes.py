"""GPU parity of the bit-plane layout decode and the layout converter
against the CPU oracle.

Tolerance: 0 bits.  The plane decode must produce exactly the oracle's
message stream and error positions for the same received words; the
converter must produce exactly the CPU re-arrangement of the bits.
"""
import numpy as np
import pytest

import oracle
import paper_1412_6862_amd as hm
import synth
from _inputs import received_words, to_device, to_host_u8, to_planes

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 2047, 2048, 2049, 4096 + 31, 20000]


def _decode_planes(planes_np, pw, n_cw, r, device, errpos=True):
    import torch

    pl = torch.from_numpy(np.ascontiguousarray(planes_np).reshape(-1).view(np.int64)).to(device)
    data, ep = hm.decode_planes(pl, pw, n_cw, r, errpos=errpos)
    torch.cuda.synchronize()
    return to_host_u8(data), (to_host_u8(ep) if errpos else None)


@pytest.mark.parametrize("r", [3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_cw", SIZES)
def test_planes_parity_ragged_sizes(gpu_device, r, n_cw):
    y = received_words(synth.workload_seed("gpu-planes", r, n_cw), n_cw, r, p_single=0.3, p_double=0.1)
    d_ref, e_ref = oracle.decode(y, r)
    d, e = _decode_planes(to_planes(y, n_cw, r), (n_cw + 63) // 64, n_cw, r, gpu_device)
    assert np.array_equal(d, d_ref) and np.array_equal(e, e_ref)


@pytest.mark.parametrize("r", [3, 5, 7])
def test_planes_parity_error_rates_padding_and_stride(gpu_device, r):
    n_cw = 70000
    for p in synth.PLAIN_ERROR_RATES:
        y = received_words(synth.workload_seed("gpu-planes-rates", r, str(p)), n_cw, r, p_single=p)
        d_ref, e_ref = oracle.decode(y, r)
        pw = (n_cw + 63) // 64 + 5          # planes further apart than needed
        planes = to_planes(y, n_cw, r, pw)
        # bits past n_cw in the last plane word are ignored
        tail = np.uint64(~((1 << (n_cw % 64)) - 1) & ((1 << 64) - 1))
        planes[:, n_cw // 64] |= tail
        planes[:, n_cw // 64 + 1:] = np.uint64(0xDEADBEEFDEADBEEF)
        d, e = _decode_planes(planes, pw, n_cw, r, gpu_device)
        assert np.array_equal(d, d_ref) and np.array_equal(e, e_ref), p
    d, e = _decode_planes(planes, pw, n_cw, r, gpu_device, errpos=False)
    assert np.array_equal(d, d_ref) and e is None


@pytest.mark.parametrize("r", [3, 4, 5, 6, 7])
def test_planes_unaligned_outputs_and_canaries(gpu_device, r):
    import torch

    n_cw = 5000 + 17
    y = received_words(synth.workload_seed("gpu-planes-align", r), n_cw, r, p_single=0.5)
    d_ref, e_ref = oracle.decode(y, r)
    pl = torch.from_numpy(to_planes(y, n_cw, r).reshape(-1).view(np.int64)).to(gpu_device)
    nb = hm.hamming_data_bytes(n_cw, r)
    big = torch.full((nb + 64,), 0x5A, dtype=torch.uint8, device=gpu_device)
    ep = torch.full((n_cw + 64,), 0xA5, dtype=torch.uint8, device=gpu_device)
    data = big[8:8 + nb]                      # 8-byte but not 16-byte aligned
    e = ep[3:3 + n_cw]                        # unaligned errpos
    hm.hamming_decode_planes(pl, (n_cw + 63) // 64, n_cw, r, data, e)
    torch.cuda.synchronize()
    b = to_host_u8(big)
    assert np.array_equal(b[8:8 + nb], d_ref) and (b[:8] == 0x5A).all() and (b[8 + nb:] == 0x5A).all()
    x = to_host_u8(ep)
    assert np.array_equal(x[3:3 + n_cw], e_ref) and (x[:3] == 0xA5).all() and (x[3 + n_cw:] == 0xA5).all()


@pytest.mark.parametrize("r", [3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_cw", [1, 33, 2049, 20000])
def test_to_planes_matches_cpu_rearrangement(gpu_device, r, n_cw):
    import torch

    y = received_words(synth.workload_seed("gpu-to-planes", r, n_cw), n_cw, r, p_single=0.3)
    planes, pw = hm.to_planes(to_device(y, gpu_device), r)
    torch.cuda.synchronize()
    got = planes.cpu().numpy().view(np.uint64).reshape((1 << r) - 1, pw)
    assert np.array_equal(got, to_planes(y, n_cw, r))


@pytest.mark.parametrize("r", [3, 5, 6, 7])
@pytest.mark.parametrize("n_cw", [2047, 2048, 2049, 8192 + 33, 16384])
@pytest.mark.parametrize("spare", [0, 1])
def test_to_planes_tiles_lines_and_canaries(gpu_device, r, n_cw, spare):
    """Around the converter's 2048-codeword tiles, planes on whole 128-byte
    lines (spare = 0) and off them, from codewords at an odd word; plane words
    past the packet keep their contents."""
    import torch

    y = received_words(synth.workload_seed("gpu-to-planes-tiles", r, n_cw), n_cw, r, p_single=0.3)
    pw = ((n_cw + 63) // 64 + 15) // 16 * 16 + 16 + spare
    N = (1 << r) - 1
    raw = torch.full((N * pw + 16,), 0x5A5A5A5A5A5A5A5A, dtype=torch.int64, device=gpu_device)
    start = (-(raw.data_ptr() // 8)) % 16 + spare
    arena = torch.zeros(y.size + 1, dtype=torch.int64, device=gpu_device)
    arena[1:] = to_device(y, gpu_device)
    hm.hamming_to_planes(arena[1:], n_cw, r, raw[start:], pw)
    torch.cuda.synchronize()
    got = raw.cpu().numpy()
    body = got[start:start + N * pw].view(np.uint32).reshape(N, 2 * pw)
    ref = to_planes(y, n_cw, r, pw).view(np.uint32).reshape(N, 2 * pw)
    dwords = (n_cw + 31) // 32
    assert np.array_equal(body[:, :dwords], ref[:, :dwords])
    assert (body[:, dwords:] == 0x5A5A5A5A).all()
    outside = np.concatenate([got[:start], got[start + N * pw:]])
    assert (outside == 0x5A5A5A5A5A5A5A5A).all()


@pytest.mark.parametrize("r,n_cw", [(3, 1 << 26), (5, 1 << 26), (7, 1 << 25)])
def test_planes_full_size_equals_plain_decode_and_oracle_samples(gpu_device, r, n_cw):
    """Full-size packets: the plane decode equals the plain decode of the
    same received words byte for byte, and sampled slices equal the oracle."""
    import torch

    seed = synth.workload_seed("gpu-planes-full", r)
    cw = hm.encode(synth.message_stream_torch(seed, n_cw, r, gpu_device), n_cw, r)
    cw ^= synth.flip_masks_torch(seed, n_cw, r, 0.1, gpu_device)
    d_plain, e_plain = hm.decode(cw, r)
    planes, pw = hm.to_planes(cw, r)
    d, e = hm.decode_planes(planes, pw, n_cw, r)
    torch.cuda.synchronize()
    assert torch.equal(d, d_plain) and torch.equal(e, e_plain)
    k = hm.hamming_message_bits(r)
    wpc = hm.words_per_codeword(r)
    for first in (0, n_cw // 3 * 64 // 64, n_cw - 64):
        first -= first % 64
        y = cw[first * wpc:(first + 64) * wpc].cpu().numpy().view(np.uint64)
        d_ref, e_ref = oracle.decode(y, r)
        got = d[first * k // 8:first * k // 8 + d_ref.size].cpu().numpy()
        assert np.array_equal(got, d_ref) and np.array_equal(e[first:first + 64].cpu().numpy(), e_ref)


@pytest.mark.parametrize("r,n_cw", [(3, 2049), (6, 33 * 32 - 5), (7, 1)])
@pytest.mark.parametrize("how", ["stream", "pointer", "null"])
def test_to_planes_on_a_stream_of_its_own_is_whole_when_that_stream_is_done(gpu_device, r, n_cw, how):
    """An odd count of 32 codewords leaves half of each plane's last word to a
    clear, which belongs to the stream that the call names: with torch's current
    stream still busy, and recycled memory that holds other bits, the planes are
    complete once the named stream is."""
    import torch

    assert (n_cw + 31) // 32 % 2
    y = received_words(synth.workload_seed("gpu-to-planes-stream", r, n_cw), n_cw, r, p_single=0.3)
    want = to_planes(y, n_cw, r)
    cw = to_device(y, gpu_device)
    current, other = torch.cuda.Stream(), torch.cuda.Stream()
    stream = {"stream": other, "pointer": other.cuda_stream, "null": 0}[how]
    waited = torch.cuda.default_stream() if how == "null" else other
    torch.cuda.synchronize()
    with torch.cuda.stream(current):
        old = torch.full((want.size,), 0x5A5A5A5A5A5A5A5A, dtype=torch.int64, device=gpu_device)
        del old
        current.synchronize()
        torch.cuda._sleep(2000000)
        planes, pw = hm.to_planes(cw, r, stream=stream)
        assert torch.cuda.current_stream() == current
    waited.synchronize()
    with torch.cuda.stream(waited):
        first = planes.cpu().numpy().view(np.uint64).reshape(want.shape)
    torch.cuda.synchronize()
    last = planes.cpu().numpy().view(np.uint64).reshape(want.shape)
    assert pw == want.shape[1] and np.array_equal(first, want) and np.array_equal(last, want)
