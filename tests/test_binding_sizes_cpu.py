"""Output sizes in the Python binding: the tensor that ``decode``,
``decode_planes`` and ``Server.result`` size for a call has exactly the bytes
that the library writes (``hamming_data_bytes``), for every integer type that
the entry points take and past the ends of their ranges."""
import types

import numpy as np
import pytest
import torch

import paper_1412_6862_amd as hm

COUNTS = [0, 1, 63, 64, 1000, 80_000_000, hm.HAMMING_MAX_CODEWORDS, hm.HAMMING_MAX_CODEWORDS + 1, 1 << 60,
          (1 << 64) + 5, -1]


@pytest.mark.parametrize("kind", [int, np.int8, np.uint8, np.int32, np.uint32, np.int64, np.uint64])
def test_message_stream_bytes_is_what_the_library_writes(kind):
    for r in (2, 3, 4, 5, 6, 7, 8):
        for n in COUNTS:
            want = hm.hamming_data_bytes(n, r)
            assert hm._message_stream_bytes(n, kind(r)) == want, (n, r)
            if kind is not int and not np.iinfo(kind).min <= n <= np.iinfo(kind).max:
                continue
            got = hm._message_stream_bytes(kind(n), r)
            assert got == want and type(got) is int, (n, r)
            assert hm._message_stream_bytes(kind(n), kind(r)) == want, (n, r)


@pytest.mark.parametrize("kind,n_cw", [(np.int8, 127), (np.uint8, 200), (np.int32, 1000), (np.uint64, 1000), (int, 1000)])
@pytest.mark.parametrize("r", [3, 6, 7])
def test_encode_allocates_every_codeword(monkeypatch, kind, n_cw, r):
    got = {}
    messages = types.SimpleNamespace(is_cuda=True, device="cpu", contiguous=lambda: None)
    monkeypatch.setattr(hm, "hamming_encode", lambda msg, n, r, out, stream=None: got.update(n=int(n), out=out))
    out = hm.encode(messages, kind(n_cw), r)
    assert out is got["out"] and got["n"] == n_cw and out.numel() == n_cw * (2 if r == 7 else 1)


@pytest.mark.parametrize("kind", [int, np.int8, np.uint8, np.int32, np.uint64])
@pytest.mark.parametrize("r", [3, 6, 7])
def test_to_planes_allocates_every_plane(monkeypatch, kind, r):
    monkeypatch.setattr(hm, "hamming_to_planes", lambda cw, n, r, planes, pw, stream=None: None)
    n_cw = 640
    planes, pw = hm.to_planes(torch.zeros(n_cw * (2 if r == 7 else 1), dtype=torch.int64), kind(r))
    assert pw == 10 and planes.numel() == ((1 << r) - 1) * 10


@pytest.mark.parametrize("kind", [int, np.int8, np.uint8, np.int32, np.uint64])
def test_server_result_views(kind):
    server = types.SimpleNamespace(output=torch.arange(2000) % 251)
    data, errpos = hm.Server.result(server, types.SimpleNamespace(data_offset=16, errpos_offset=240), 6, kind(100))
    assert torch.equal(data, server.output[16:16 + 720]) and torch.equal(errpos, server.output[240:340])
