// Host side of the batched decode: how many launches a batch takes and how
// it is read, and of a planned batch (see PlannedBatch in batch.h) the coarse
// tile-to-packet map built from the packets' tile prefix sums.  Host code only.
#pragma once

#include <stdint.h>

namespace hm {

// How a batch is launched (launch_batch), by the packets that the caller's
// arguments allow and the workgroups of one chunk per wave that it fills, before
// any cap on the grid.  A launch after another costs 4-5 us (the gap and the ramp),
// so short batches take fewer; what they pay for it, they pay per workgroup and per
// chunk, whatever its bytes (and also when a cap of 4096 makes waves loop: 256
// packets, 140 MB, 51 us in one launch, 48 in two):
//  * one launch, every workgroup planning for itself, up to kOnePackets packets
//    and kOneBlocks workgroups (the planning, about 2 us, is paid once per
//    resident workgroup: 200 packets, 34 MB: 14 us against 16 us with two launches
//    and 21 with four; 256 packets, 140 MB: 41 against 35 in 8700 workgroups, but
//    60 against 61 in 1100, chunks of 8 tiles; 400 MB 126 against 135);
//  * two, plan with a coarse map and decode, up to kMapPackets packets and
//    kMapBlocks workgroups (1000 packets, 47 MB: 19.5 against 24 us; 400 MB in
//    chunks of 8 tiles 131 against 134), above which the decode's longer lookup
//    outweighs a launch (2000 packets, 3.7 GB: decode 618-655 against 584-631 us
//    with the fine map);
//  * three, plan, fine map and decode.
enum class BatchForm { one, two, three };

constexpr uint32_t kOnePackets = 256;
constexpr uint64_t kOneBlocks = 4096;
constexpr uint32_t kMapPackets = 1024;
constexpr uint64_t kMapBlocks = 16384;

constexpr BatchForm batch_form(uint32_t max_packets, uint64_t blocks)
{
    if (max_packets <= kOnePackets && blocks <= kOneBlocks) return BatchForm::one;
    return max_packets <= kMapPackets && blocks <= kMapBlocks ? BatchForm::two : BatchForm::three;
}

// Whether a one- or two-launch batch of at most in_bytes is read with ordinary
// loads, which the caches answer where they hold the packets, or with streaming
// loads, as every batch of three launches.  How many workgroups share the bytes is
// no part of it: 256 packets decoded in one launch of chunks of 8 tiles, ordinary
// against streaming loads: 60 MB repeated 21.6 against 24.2 us, just written 21.7
// against 21.9, from HBM 26.3 against 25.0; 100 MB just written 35.2 against 31.8,
// from HBM 40.9 against 38.6; 240 MB 87.7 against 72.5 and 86.9 against 81.9.
constexpr uint64_t kBatchCachedBytes = uint64_t(64) << 20;
constexpr bool batch_reads_cached(uint64_t in_bytes) { return in_bytes <= kBatchCachedBytes; }

// Input bytes of the largest batch that the arguments allow: the arena, or the
// caller's bound on the codewords (0: none) at 16 bytes each.
constexpr uint64_t batch_input_bytes(uint64_t cw_words, uint64_t max_codewords)
{
    const uint64_t words = max_codewords && max_codewords < cw_words / 2 ? 2 * max_codewords : cw_words;
    return words > (~uint64_t(0) >> 3) ? ~uint64_t(0) : 8 * words;
}

// Coarse-map entries a host plan of n packets may use.
inline uint64_t planned_coarse_capacity(uint32_t n) { return 2ull * n + 64; }

// Smallest g with ceil(total / 2^g) <= planned_coarse_capacity(n).
inline uint32_t planned_coarse_log2(uint64_t total, uint32_t n)
{
    const uint64_t cap = planned_coarse_capacity(n);
    uint32_t g = 0;
    while ((total >> g) >= cap) ++g;
    return g;
}

// Fill coarse[j] with the packet holding tile j << g, for every j below
// ceil(ts[n] / 2^g); ts[0..n] is the exclusive prefix sum of the packets'
// tile counts (packets without tiles included).  Entry j gets the first
// packet p, in order, with (j << g) < ts[p + 1]; every earlier packet ends at
// or before that tile, so ts[p] <= (j << g) as well.  Returns the entries.
inline uint64_t plan_coarse_map(const uint64_t* ts, uint32_t n, uint32_t g, uint32_t* coarse)
{
    const uint64_t entries = (ts[n] + (uint64_t(1) << g) - 1) >> g;
    uint64_t j = 0;
    for (uint32_t p = 0; p < n && j < entries; ++p)
        while (j < entries && (j << g) < ts[p + 1]) coarse[j++] = p;
    return entries;
}

}  // namespace hm
