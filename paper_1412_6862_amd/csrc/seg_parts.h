// The part form of the segmented-packet kernels (segmented.hip): how a packet
// is dealt to a group of lanes, and the bit work of one 128-position window on
// 32-bit registers.  Pure functions, compiled for the device and for the host,
// so that host code can run a whole packet through them.
//
// Every segment is cut into the same number of parts, a part is a few
// consecutive windows, and a lane owns one part of one segment.  It therefore
// folds its windows into a syndrome in registers, without a word of LDS, until
// its part ends.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hm {

// Bits sh..sh+31 (sh taken mod 32) of the 64-bit value hi:lo.
__host__ __device__ inline uint32_t align32(uint32_t hi, uint32_t lo, uint32_t sh)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_alignbit(hi, lo, sh);
#else
    return uint32_t(((uint64_t(hi) << 32) | lo) >> (sh & 31u));
#endif
}

// x / y for x < 2^16 and 1 <= y < 2^16 without the generic division: the
// quotient estimate is at most one off, and is put right on whole numbers.
__host__ __device__ inline uint32_t small_div(uint32_t x, uint32_t y)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t q = uint32_t(float(x) * __builtin_amdgcn_rcpf(float(y)));
#else
    uint32_t q = uint32_t(float(x) * (1.0f / float(y)));
#endif
    q -= q * y > x ? 1u : 0u;
    q += (q + 1u) * y <= x ? 1u : 0u;
    return q;
}

// How a packet of t segments of at most v windows is dealt to `group` lanes:
// lane l takes part l % parts of segment l / parts, windows [part * len,
// part * len + len).  inv divides a lane index by parts.
struct Parts {
    uint32_t parts, len, inv;

    __host__ __device__ uint32_t segment(uint32_t lane) const { return (lane * inv) >> 16; }
};

// Needs 1 <= t <= group <= 64.
__host__ __device__ inline Parts make_parts(uint32_t t, uint32_t v, uint32_t group)
{
    Parts p;
    p.parts = small_div(group, t);
    p.len = small_div(v + p.parts - 1u, p.parts);
    // ceil(2^16 / parts): (lane * inv) >> 16 = lane / parts for lane < 64, as
    // the excess over lane / parts is below 64 / 2^16 < 1 / parts
    p.inv = small_div(65535u, p.parts) + 1u;
    return p;
}

// Keeps bits 0..top of a window of four dwords (top < 0: none, top >= 127: all).
__host__ __device__ inline void mask_window(uint32_t (&x)[4], int32_t top)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int32_t c = top + 1 - 32 * k;                 // bits to keep of dword k
        c = c < 0 ? 0 : (c > 32 ? 32 : c);
        x[k] &= uint32_t((uint64_t(0xFFFFFFFFu) << c) >> 32);
    }
}

// Partial syndrome of a part: parity accumulators of its windows' dwords.
struct PartSyndrome {
    uint32_t all = 0;    // XOR of all dwords: position bits 0..4
    uint32_t odd = 0;    // XOR of dwords 1 and 3: bit 5
    uint32_t high = 0;   // XOR of dwords 2 and 3: bit 6
    uint32_t win = 0;    // XOR of the indices of the windows of odd weight: bits 7 and up

    // Folds window v (bit b of dword k = position 128v + 32k + b).
    __host__ __device__ void add(const uint32_t (&x)[4], uint32_t v)
    {
        const uint32_t f = x[0] ^ x[1] ^ x[2] ^ x[3];
        all ^= f;
        odd ^= x[1] ^ x[3];
        high ^= x[2] ^ x[3];
        win ^= (0u - (uint32_t(__builtin_popcount(f)) & 1u)) & v;
    }

    // XOR of the positions of the set bits folded so far.
    __host__ __device__ uint32_t value() const
    {
        uint32_t s = win << 7;
        s |= uint32_t(__builtin_popcount(all & 0xAAAAAAAAu)) & 1u;
        s |= (uint32_t(__builtin_popcount(all & 0xCCCCCCCCu)) & 1u) << 1;
        s |= (uint32_t(__builtin_popcount(all & 0xF0F0F0F0u)) & 1u) << 2;
        s |= (uint32_t(__builtin_popcount(all & 0xFF00FF00u)) & 1u) << 3;
        s |= (uint32_t(__builtin_popcount(all & 0xFFFF0000u)) & 1u) << 4;
        s |= (uint32_t(__builtin_popcount(odd)) & 1u) << 5;
        s |= (uint32_t(__builtin_popcount(high)) & 1u) << 6;
        return s;
    }
};

// Message index, within its segment, that position 128v would have if it were
// a message position (v >= 1): 128v minus the floor(log2 v) + 8 checksum
// positions below it, minus one.  Position 128v + q then carries message bit
// run_base(v) + q, except that 128v itself is a checksum position when v is a
// power of two; its index is then the last one of the run before.
__host__ __device__ inline uint32_t run_base(uint32_t v)
{
    return 128u * v - (31u - uint32_t(__builtin_clz(v | 1u))) - 9u;
}

__host__ __device__ inline uint32_t is_pow2_window(uint32_t v) { return (v & (v - 1u)) == 0u ? 1u : 0u; }

// Window 0 (positions 0..127) to its 120 message bits, compacted.
__host__ __device__ inline void compact_head(uint32_t (&x)[4])
{
    const uint32_t h = ((x[0] >> 3) & 0x1u) | ((x[0] >> 4) & 0xEu) | ((x[0] >> 5) & 0x7F0u) |
                       ((x[0] >> 6) & 0x3FFF800u);                      // positions 3, 5-7, 9-15, 17-31
    const uint32_t x1 = x[1], x2 = x[2], x3 = x[3];
    x[0] = h | ((x1 << 25) & 0xFC000000u);                              // positions 33-63
    x[1] = (x1 >> 7) | ((x2 << 24) & 0xFE000000u);                      // positions 65-127
    x[2] = (x2 >> 8) | (x3 << 24);
    x[3] = x3 >> 8;
}

// The inverse: 120 message bits (bits past them ignored) to their positions
// in window 0, checksum positions 0.
__host__ __device__ inline void expand_head(uint32_t (&m)[4])
{
    const uint32_t m0 = m[0], m1 = m[1], m2 = m[2], m3 = m[3];
    m[0] = ((m0 & 0x1u) << 3) | ((m0 & 0xEu) << 4) | ((m0 & 0x7F0u) << 5) | ((m0 & 0x3FFF800u) << 6);
    m[1] = ((m0 >> 25) & 0x7Eu) | (m1 << 7);
    m[2] = ((m1 >> 24) & 0xFEu) | (m2 << 8);
    m[3] = (m2 >> 24) | (m3 << 8);
}

// A staged run lies in LDS in blocks of 32 dwords, each followed by room for four
// more: while packets are read these hold the first four dwords of the next block,
// and while results are built they collect what is ORed past a block's end, which
// is merged into the next block at last.  The five dwords of a window are thus
// consecutive wherever it starts, and lanes whose windows lie a multiple of 32
// dwords apart, as those of segments and packets of about 1024 bits or a multiple
// do, meet 4 dwords apart in the banks instead of all in one.
constexpr uint32_t kBlockDwords = 32, kBlockRoom = 4;

// LDS dword of dword a of the run's area; with R < kBlockRoom, dword a is also at
// block_at(a) - kBlockRoom if a % kBlockDwords == R (the room of the block before).
__host__ __device__ inline uint32_t block_at(uint32_t a) { return a + a / kBlockDwords * kBlockRoom; }

// LDS dwords of an area of `dwords` dwords, the last block's room included.
__host__ __device__ constexpr uint32_t block_area(uint32_t dwords)
{
    return dwords + (dwords + kBlockDwords - 1u) / kBlockDwords * kBlockRoom;
}

// Dwords of the largest area that `lds` LDS dwords hold: block_area(it) <= lds.
__host__ __device__ constexpr uint32_t block_capacity(uint32_t lds)
{
    return lds < kBlockRoom ? 0u : (lds - kBlockRoom) * kBlockDwords / (kBlockDwords + kBlockRoom);
}

// A window to be placed at bit `at` (>= 0) of a dword array: the window's bits
// go to dwords first .. first + 4, where first may be -1 (that dword then gets
// zero bits only).
struct Placed {
    int32_t first;
    uint32_t y[5];
};

__host__ __device__ inline Placed place_window(const uint32_t (&x)[4], uint32_t at)
{
    Placed p;
    p.first = int32_t(at - 1u) >> 5;
    const uint32_t sh = 0u - at;
    p.y[0] = align32(x[0], 0u, sh);
    p.y[1] = align32(x[1], x[0], sh);
    p.y[2] = align32(x[2], x[1], sh);
    p.y[3] = align32(x[3], x[2], sh);
    p.y[4] = align32(0u, x[3], sh);
    return p;
}

}  // namespace hm
