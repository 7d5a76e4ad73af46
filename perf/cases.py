"""The work that programs have the Hamming library do, as cases to be timed.

A case is a dict of plain values.  ``prepare`` puts on the GPU what a program
has in hand before a call (received codewords, messages, descriptors, the
decoder or server object it keeps), ``run`` makes one pass through the public
entry points and returns everything the pass computed, ``work`` says how many
bytes the pass cannot do without.  Packet sizes of a mixed batch come from the
case itself, contents from the seed.

Received words are what a channel delivers: uniform message bits, encoded, a
fraction of the codewords with one flipped bit at a uniform position (checksum
positions included), for Hamming(127,120) also some with two.  Every output is
bits or whole numbers, so there is no value in 64-bit floating point to hold
them against: ``exact`` gives none and outputs have to be equal.
"""
from __future__ import annotations

import math
import os
import random

import numpy as np
import torch

import paper_1412_6862_amd as hm

TUNED = os.path.join(os.path.dirname(os.path.abspath(hm.__file__)), "tuned_shapes.json")


def listed():
    return [
        # one received block of the smallest code: a latency call, most of it launch
        {"name": "decode_7_4_block", "kind": "decode", "r": 3, "n_cw": 65536, "single": 0.5, "double": 0.0},
        # an ordinary packet whose length is no multiple of anything
        {"name": "decode_15_11_packet", "kind": "decode", "r": 4, "n_cw": 1000003, "single": 0.1, "double": 0.0},
        # the dominant packet of the throughput benchmark
        {"name": "decode_63_57_large", "kind": "decode", "r": 6, "n_cw": 1 << 26, "single": 0.1, "double": 0.0},
        # two storage words per codeword, with errors beyond the code's reach
        {"name": "decode_127_120_large", "kind": "decode", "r": 7, "n_cw": 1 << 25, "single": 0.25, "double": 0.05},
        # the transmitter's half at the benchmark's size
        {"name": "encode_63_57_large", "kind": "encode", "r": 6, "n_cw": 1 << 26},
        # a handful of short packets of all codes in one call: launches and lookups count
        {"name": "batch_short", "kind": "batch", "packets": 48, "lo": 64, "span": 6.0, "mix": 1},
        # a receiver's batch: many packets of all codes, sizes over four decades
        {"name": "batch_mixed", "kind": "batch", "packets": 2000, "lo": 64, "span": 14.0, "mix": 2},
        # a burst of requests through the server, from submission to the last completion
        {"name": "serve_burst", "kind": "serve", "requests": 24, "lo": 256, "span": 10.0, "mix": 3},
        # a few long packets in the paper's own format: latency
        {"name": "seg_decode_few", "kind": "seg_decode", "packets": 64, "bytes": 2000, "t": 6},
        # the paper's packets in bulk, middle of its grid of sizes and segment counts
        {"name": "seg_decode_bulk", "kind": "seg_decode", "packets": 1 << 19, "bytes": 1200, "t": 4},
        # their transmitter
        {"name": "seg_encode_bulk", "kind": "seg_encode", "packets": 1 << 18, "bytes": 800, "t": 5},
        # received words brought into the bit-plane layout and decoded there
        {"name": "planes_31_26", "kind": "planes", "r": 5, "n_cw": (1 << 24) + 77, "single": 0.1},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "encode", "batch", "serve", "seg_decode", "seg_decode", "seg_encode",
                       "planes"])
    if kind in ("decode", "encode", "planes"):
        r = rng.randint(3, 7)
        top = (1 << 24) if kind == "planes" else (1 << 25) if r == 7 else (1 << 26)
        case = {"kind": kind, "r": r, "n_cw": _log_int(rng, 1000, top)}
        if kind != "encode":
            case["single"] = rng.choice([0.0, 0.01, 0.1, 0.5])
        if kind == "decode":
            case["double"] = rng.choice([0.0, 0.05])
        return case
    if kind == "batch":
        return {"kind": kind, "packets": _log_int(rng, 2, 2000), "lo": 64, "span": round(rng.uniform(4.0, 14.0), 2),
                "mix": rng.randrange(1 << 20)}
    if kind == "serve":
        return {"kind": kind, "requests": rng.randint(2, 28), "lo": 256, "span": round(rng.uniform(4.0, 10.0), 2),
                "mix": rng.randrange(1 << 20)}
    # the paper's range of packet sizes and segment counts; batches of up to 2^29 message bytes
    size, t = rng.randint(400, 2000), rng.randint(2, 6)
    return {"kind": kind, "packets": _log_int(rng, 1, min(1 << 19, (1 << 29) // size)), "bytes": size, "t": t}


# ---- inputs ------------------------------------------------------------------------


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _random_words(n, g):
    return torch.randint(-(1 << 63), (1 << 63) - 1, (n,), dtype=torch.int64, device="cuda", generator=g)


def _flip(cw, r, single, double, g):
    """Flip one (or two) bits of a fraction of the codewords, in place."""
    n = (1 << r) - 1
    n_cw = cw.numel() // hm.words_per_codeword(r)
    if single <= 0.0 and double <= 0.0:
        return
    u = torch.rand(n_cw, device="cuda", generator=g)
    for part, limit in ((0, single + double), (1, double)):
        if limit <= 0.0:
            continue
        pos = torch.randint(0, n, (n_cw,), dtype=torch.int64, device="cuda", generator=g)
        hit = (u < limit).to(torch.int64)
        if r < 7:
            cw ^= hit << pos
        else:
            w = cw.view(n_cw, 2)
            high = pos >> 6
            w[:, 0] ^= (hit * (1 - high)) << (pos & 63)
            w[:, 1] ^= (hit * high) << (pos & 63)


def _received(n_cw, r, single, double, g, out=None):
    """n_cw received codewords (into ``out`` when given)."""
    msg = _random_words((n_cw * hm.hamming_message_bits(r) + 63) // 64, g)
    cw = torch.empty(n_cw * hm.words_per_codeword(r), dtype=torch.int64, device="cuda") if out is None else out
    hm.hamming_encode(msg, n_cw, r, cw)
    _flip(cw, r, single, double, g)
    return cw


def _mixed_sizes(case, count, codes):
    """(r, n_cw, error rate) of each packet of a mixed batch."""
    rng = random.Random(int(case["mix"]))
    return [(rng.choice(codes), int(case["lo"] * 2.0 ** (case["span"] * rng.random())), 0.5 * rng.random())
            for _ in range(count)]


def _packed(sizes, g):
    """The packets end to end in one arena, and each one's first word."""
    words = [n * hm.words_per_codeword(r) for r, n, _ in sizes]
    offs = np.concatenate([[0], np.cumsum(words)]).astype(np.int64)
    arena = torch.empty(int(offs[-1]), dtype=torch.int64, device="cuda")
    for (r, n, p), a, w in zip(sizes, offs, words):
        _received(n, r, p, 0.0, g, arena[int(a):int(a) + w])
    return arena, offs[:-1]


def _segmented(case, g, received):
    b = hm.SegmentedBatch(case["packets"], case["bytes"], case["t"])
    b.msg.copy_(_random_words(b.msg.numel(), g))
    if case["bytes"] % 8:
        b.msg.view(-1, b.msg_stride)[:, -1] &= (1 << (8 * (case["bytes"] % 8))) - 1
    if received:
        b.encode()
        b.msg.zero_()
        enc = b.enc.view(case["packets"], b.enc_stride)
        k, r, _ = hm.hamming_seg_layout(case["bytes"], case["t"])
        start = 0
        for n in (x + y for x, y in zip(k, r)):
            u = torch.rand(case["packets"], device="cuda", generator=g)
            for limit in (0.35, 0.05):         # one flip in 0.3 of the segments, two in 0.05
                pos = start + torch.randint(0, n, (case["packets"], 1), dtype=torch.int64, device="cuda", generator=g)
                bit = (u < limit).to(torch.int64)[:, None] << (pos & 63)
                enc.scatter_(1, pos >> 6, enc.gather(1, pos >> 6) ^ bit)
            start += n
    return b


def prepare(case, seed):
    hm.hamming_tune_load(TUNED)      # the launch shapes that ship with the library
    g = _generator(seed)
    kind = case["kind"]
    if kind in ("decode", "planes"):
        return {"case": case, "cw": _received(case["n_cw"], case["r"], case["single"], case.get("double", 0.0), g)}
    if kind == "encode":
        return {"case": case, "msg": _random_words((case["n_cw"] * hm.hamming_message_bits(case["r"]) + 63) // 64, g)}
    if kind == "batch":
        sizes = _mixed_sizes(case, case["packets"], (3, 4, 5, 6, 7))
        arena, offs = _packed(sizes, g)
        descs = np.zeros(len(sizes), dtype=hm.packet_dtype())
        descs["in_word_off"] = offs
        descs["r"] = [s[0] for s in sizes]
        descs["n_cw"] = [s[1] for s in sizes]
        batch = hm.BatchDecoder(arena, len(sizes))
        batch.set_packets(descs)
        batch.data.zero_()           # the alignment gaps between packets are never written
        batch.errpos.zero_()
        return {"case": case, "batch": batch, "codewords": int(descs["n_cw"].sum())}
    if kind == "serve":
        sizes = _mixed_sizes(case, case["requests"], (4, 5, 6, 7))
        pool, offs = _packed(sizes, g)
        server = hm.Server(pool, slots=4, max_batch_packets=4096, max_batch_codewords=1 << 25,
                           output_pool_bytes=256 << 20, max_queue=4096)
        return {"case": case, "server": server, "live": [],
                "requests": [(int(o), n, r) for (r, n, _), o in zip(sizes, offs)]}
    return {"case": case, "batch": _segmented(case, g, kind == "seg_decode")}


# ---- one pass ----------------------------------------------------------------------


def _serve(state):
    """Release the last burst's outputs, submit a burst, wait for its completions."""
    server, requests = state["server"], state["requests"]
    for rid in state["live"]:
        server.release(rid)
    first = None
    for off, n, r in requests:
        rid = server.submit(off, n, r)
        first = rid if first is None else first
    done = [None] * len(requests)
    left = len(requests)
    while left:
        server.progress()
        for c in server.poll(64):
            done[c.request_id - first] = c
            left -= 1
    state["live"] = list(range(first, first + len(requests)))
    return [server.result(c, r, n) for c, (_, n, r) in zip(done, requests)]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "decode":
        return hm.decode(state["cw"], case["r"])
    if kind == "encode":
        return hm.encode(state["msg"], case["n_cw"], case["r"])
    if kind == "batch":
        b = state["batch"]
        b.decode(max_codewords=state["codewords"])
        return [b.data, b.errpos, b.status]
    if kind == "serve":
        return _serve(state)
    if kind == "planes":
        planes, stride = hm.to_planes(state["cw"], case["r"])
        data, errpos = hm.decode_planes(planes, stride, case["n_cw"], case["r"])
        return [planes, data, errpos]
    b = state["batch"]
    if kind == "seg_decode":
        b.decode()
        return [b.msg, b.syndromes, b.status]
    b.encode()
    return b.enc


# ---- what a pass cannot do without ----------------------------------------------------


def _message_bytes(n_cw, r):
    return (n_cw * ((1 << r) - 1 - r) + 63) // 64 * 8


def _decode_bytes(n_cw, r):
    return n_cw * (16 if r == 7 else 8) + _message_bytes(n_cw, r) + n_cw


def work(case):
    kind = case["kind"]
    if kind == "decode":
        moved = _decode_bytes(case["n_cw"], case["r"])
    elif kind == "encode":
        moved = case["n_cw"] * (16 if case["r"] == 7 else 8) + _message_bytes(case["n_cw"], case["r"])
    elif kind == "batch":
        moved = sum(_decode_bytes(n, r) + 44 for r, n, _ in _mixed_sizes(case, case["packets"], (3, 4, 5, 6, 7)))
    elif kind == "serve":
        moved = sum(_decode_bytes(n, r) for r, n, _ in _mixed_sizes(case, case["requests"], (4, 5, 6, 7)))
    elif kind == "planes":
        n, r = case["n_cw"], case["r"]
        planes = ((1 << r) - 1) * ((n + 63) // 64) * 8
        moved = n * (16 if r == 7 else 8) + 2 * planes + _message_bytes(n, r) + n
    else:
        _, _, bits = hm.hamming_seg_layout(case["bytes"], case["t"])
        moved = case["packets"] * ((bits + 7) // 8 + 32 + case["bytes"])
        if kind == "seg_decode":
            moved += case["packets"] * (2 * case["t"] + 1)
    return {"bytes": moved, "flops": 0}


def exact(case, seed):
    return None
