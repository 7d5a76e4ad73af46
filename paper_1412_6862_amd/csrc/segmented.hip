// Segmented packets (Sec. II, Fig. 1): a packet of M message bytes travels
// as t shortened Hamming segments H_1..H_t laid end to end as one bit
// string; each segment is checked and corrected on its own and the recovered
// message segments are merged back into the M-byte packet.  The checksum of a
// segment is the XOR over its index sets (Sec. III.A, III.C, Algorithm 1).
//
// A group of threads per packet (part of a wave, a wave or a workgroup), in one
// of two forms.  A wave whose packets lie end to end (of one shape or of several),
// or of one shape at one stride, takes the part form (below, at its kernels);
// every other wave, batches of packets under 192 bytes and the workgroup per packet
// take the window form:
//
// The 128-position windows of all segments form one flat list dealt to the
// threads.  Decoding, a thread reads each of its windows once from HBM (an
// unaligned three-word span), folds it into its partial syndrome of the
// segment and ORs the window's message bits (one run of consecutive message
// indices per window) into the packet's message buffer in LDS; the segment
// owners then finish the syndromes and flip the one message bit a
// correctable error hits, and the buffer is stored.  Encoding runs the same
// walk the other way: a thread reads the message run of each window, places
// it at the window's positions, folds it into the partial syndrome and ORs it
// into the packet's encoded buffer in LDS; the owners set checksum position
// 2^j to bit j of the syndrome.  Segment offsets are closed-form (message
// sizes take two values), so no lookup table is read.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hamming.h"
#include "launch.h"
#include "seg_bits.h"
#include "seg_parts.h"
#include "tile.h"

using hm::block_area;
using hm::block_at;
using hm::block_capacity;
using hm::funnel128;
using hm::head_expand;
using hm::head_message;
using hm::kBlockDwords;
using hm::kBlockRoom;
using hm::mask_top;
using hm::run_start;
using hm::small_div;
using hm::u32x4;
using hm::u32x4a8;
using hm::wave_sync;

namespace {

constexpr uint32_t kSegWaves = 4;                          // waves per block

// Encoded words of the longest packet of at most max_msg_bytes message
// bytes, plus a word in front (stream bit -1, where the first window of the
// packet starts) and two behind (a window ORed in at a bit offset touches
// three words).
__host__ __device__ inline uint32_t enc_slice_words(uint32_t max_msg_bytes)
{
    return (8u * max_msg_bytes + 16u * HAMMING_SEG_MAX_T + 63u) / 64u + 3u;
}

// Message words of the longest packet plus three (a message run ORed in at a
// bit offset touches up to three words) plus one (the buffer is cleared in
// pairs of words).
__host__ __device__ inline uint32_t msg_slice_words(uint32_t max_msg_bytes)
{
    return (max_msg_bytes + 7u) / 8u + 4u;
}

// Checksum bits of a shortened segment with k >= 1 message bits: the
// smallest r >= 2 with 2^r - 1 - r >= k.  With b the bit length of k, r is b,
// or b + 1 when 2^b - 1 - b < k (2^(b-1) - b < k always rules out b - 1).
__host__ __device__ inline uint32_t seg_checksum_bits(uint32_t k)
{
    const uint32_t b = 32u - uint32_t(__builtin_clz(k));
    const uint32_t r = b + (((1u << b) - 1u - b) < k ? 1u : 0u);
    return r < 2 ? 2 : r;
}

// Segment layout of one packet in closed form.  The first `rem` segments
// carry q+1 message bits and nA positions, the others q bits and nB
// positions, so every offset is a product and a min.  vA and vB count the
// 128-position windows of a segment (window v = positions 128v..128v+127,
// position 0 included so that window 0 is aligned like the others).
struct Layout {
    uint32_t t, q, rem, nA, nB, vA, vB, total;

    __device__ uint32_t K(uint32_t i) const { return i * q + min(i, rem); }            // first message bit
    __device__ uint32_t o(uint32_t i) const { return i * nB + min(i, rem) * (nA - nB); }  // first stream bit
    __device__ uint32_t n(uint32_t i) const { return i < rem ? nA : nB; }
    __device__ uint32_t windows() const { return rem * vA + (t - rem) * vB; }
};

// Validates the packet shape; returns false for one this launch cannot take.
__device__ __forceinline__ bool make_layout(uint32_t msg_bytes, uint32_t t, uint32_t max_msg_bytes, Layout& L)
{
    if (t < 1 || t > HAMMING_SEG_MAX_T || msg_bytes < 1 || msg_bytes > max_msg_bytes || 8u * msg_bytes < t) return false;
    const uint32_t bits = 8u * msg_bytes;
    L.t = t;
    L.q = small_div(bits, t);                                  // bits <= 2^15
    L.rem = bits - L.q * t;
    if (L.q + (L.rem ? 1u : 0u) > HAMMING_SEG_MAX_K) return false;
    L.nA = L.q + 1 + seg_checksum_bits(L.q + 1);
    L.nB = L.q + seg_checksum_bits(L.q);
    L.vA = L.nA / 128 + 1;
    L.vB = L.nB / 128 + 1;
    L.total = L.o(t);
    return true;
}

// A thread's position in the flat list of windows: segment i, window v of
// it (nv windows), and the segment's first stream bit, positions and first
// message bit.
struct WindowWalk {
    uint32_t i, v, nv, o, n, K;

    __device__ WindowWalk(const Layout& Lo, uint32_t first)
        : i(0), v(first), nv(Lo.rem > 0 ? Lo.vA : Lo.vB), o(0), n(Lo.n(0)), K(0) {}

    // Moves forward to the segment holding window v (a window past the
    // packet's last one stays in the last segment; it is never used).
    __device__ void settle(const Layout& Lo)
    {
        while (v >= nv && i + 1 < Lo.t) {
            v -= nv;
            ++i;
            nv = i < Lo.rem ? Lo.vA : Lo.vB;
            o = Lo.o(i);
            n = Lo.n(i);
            K = Lo.K(i);
        }
    }
};

// ORs 128 bits into a word array at word bq, bit bs (three LDS atomics:
// neighbouring threads' runs share the boundary words).
__device__ __forceinline__ void or128(uint64_t* W, uint32_t bq, uint32_t bs, uint64_t x0, uint64_t x1)
{
    atomicOr(reinterpret_cast<unsigned long long*>(&W[bq]), x0 << bs);
    atomicOr(reinterpret_cast<unsigned long long*>(&W[bq + 1]), ((x0 >> 1) >> (63u - bs)) | (x1 << bs));
    atomicOr(reinterpret_cast<unsigned long long*>(&W[bq + 2]), (x1 >> 1) >> (63u - bs));
}

// Folds window v (bit q of (x0, x1) = position 128v + q) into a partial
// syndrome: bits 0..5 of a position are those of q mod 64 (the XOR of the
// halves), bit 6 says which half, bits 7 and up are those of v.
__device__ __forceinline__ void fold_window(uint64_t x0, uint64_t x1, uint32_t v, uint64_t& xacc, uint32_t& hacc)
{
    const uint64_t f = x0 ^ x1;
    xacc ^= f;
    hacc ^= ((uint32_t(__popcll(x1)) & 1u) << 6) ^ ((__popcll(f) & 1u) ? 128u * v : 0u);
}

// Syndrome of a segment from the XOR X of its 64-position halves and the
// high part H: bits 0..4 of a position are shared by bits q and q+32 of a
// half, so those five parities are taken on the XOR of its 32-bit halves; bit
// 5 is the parity of the upper 32 bits.
__device__ __forceinline__ uint32_t fold_syndrome(uint64_t x, uint32_t h)
{
    const uint32_t hi = uint32_t(x >> 32), f = uint32_t(x) ^ hi;
    uint32_t v = h;
    v ^= __popc(f & 0xAAAAAAAAu) & 1u;
    v ^= (__popc(f & 0xCCCCCCCCu) & 1u) << 1;
    v ^= (__popc(f & 0xF0F0F0F0u) & 1u) << 2;
    v ^= (__popc(f & 0xFF00FF00u) & 1u) << 3;
    v ^= (__popc(f & 0xFFFF0000u) & 1u) << 4;
    v ^= (__popc(hi) & 1u) << 5;
    return v;
}

// Adds a thread's partial syndrome of segment i to the segment's accumulators.
// Threads whose windows cancelled (or that had none) skip the LDS atomics,
// which all threads of a segment aim at the same two addresses.
__device__ __forceinline__ void flush_partial(uint64_t* X, uint32_t* H, uint32_t i, uint64_t x, uint32_t h)
{
    if (x | h) {
        atomicXor(reinterpret_cast<unsigned long long*>(&X[i]), x);
        atomicXor(&H[i], h);
    }
}

// Barrier of the threads that work on one packet: part of a wave or one wave
// (the wave runs in lockstep), or the workgroup.
template <uint32_t GROUP>
__device__ __forceinline__ void group_sync()
{
    if constexpr (GROUP <= 64) {
        wave_sync();
    } else {
        __syncthreads();
    }
}

// Decoding pass over the windows of a packet (thread gl takes flat windows
// gl, gl + GROUP, ...; it issues the loads of BATCH windows before it uses
// the first).  Each window is read from the encoded stream src as three
// words, folded into the thread's partial syndrome of its segment (flushed
// to X/H in LDS when the thread moves on to the next segment), and its
// message run is ORed into the message buffer Mb; window 0 holds the 57 head
// bits, checksum position 64 and 63 more message bits.  Mb (mw + 3 words), X
// and H must be zero and visible on entry; the result is visible to the
// group on return.
template <uint32_t GROUP, uint32_t BATCH>
__device__ __forceinline__ void decode_windows(const uint64_t* src, uint32_t ew, const Layout& Lo, uint64_t* Mb,
                                               uint64_t* X, uint32_t* H, uint32_t gl)
{
    const uint32_t wins = Lo.windows(), last = ew - 1u;
    WindowWalk walk(Lo, gl);
    uint32_t ci = 0;              // segment of the partial syndrome in xacc/hacc
    uint64_t xacc = 0;
    uint32_t hacc = 0;
    for (uint32_t g0 = gl; g0 < wins; g0 += BATCH * GROUP) {
        uint64_t a[BATCH], b[BATCH], c[BATCH];
        int32_t qw[BATCH];
        uint32_t seg[BATCH], wd[BATCH], sh[BATCH], nn[BATCH], kk[BATCH];
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            walk.settle(Lo);
            // position 128v of segment i is stream bit s0 (-1, before the
            // packet, for the first window of segment 0)
            const int32_t s0 = int32_t(walk.o + 128u * walk.v) - 1;
            qw[u] = s0 >> 6;
            seg[u] = walk.i;
            wd[u] = walk.v;
            sh[u] = uint32_t(s0) & 63u;
            nn[u] = walk.n;
            kk[u] = walk.K;
            walk.v += GROUP;
        }
        // Unconditional loads clamped into the packet: for s0 = -1 the stray
        // bit lands on position 0, and a word past the packet supplies only
        // positions past the last segment; both are masked below.
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            a[u] = src[min(uint32_t(max(qw[u], 0)), last)];
            b[u] = src[min(uint32_t(qw[u] + 1), last)];
            c[u] = src[min(uint32_t(qw[u] + 2), last)];
        }
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            if (g0 + u * GROUP >= wins) break;
            const uint32_t v = wd[u];
            uint64_t x0, x1;
            funnel128(a[u], b[u], c[u], sh[u], x0, x1);
            mask_top(x0, x1, nn[u] - 128u * v);
            x0 &= ~uint64_t(v == 0 ? 1u : 0u);            // there is no position 0

            if (seg[u] != ci) {
                flush_partial(X, H, ci, xacc, hacc);
                ci = seg[u];
                xacc = 0;
                hacc = 0;
            }
            fold_window(x0, x1, v, xacc, hacc);

            uint32_t pw;
            const uint32_t b0 = kk[u] + run_start(v, pw);
            uint64_t c0 = (x0 >> pw) | ((x1 << 1) << (63u - pw));
            uint64_t c1 = x1 >> pw;
            if (v == 0) {
                c0 = head_message(c0) | (c1 << 57);
                c1 >>= 7;
            }
            or128(Mb, b0 >> 6, b0 & 63u, c0, c1);
        }
    }
    flush_partial(X, H, ci, xacc, hacc);
    group_sync<GROUP>();
}

// Encoding pass, the decoding pass reversed: each window's message run is
// read from the message words src (mw words; clamped reads past the packet
// supply only bits that land past the last segment's positions), placed at
// the window's positions with its checksum positions 0, folded into the
// partial syndrome, and ORed into the encoded buffer E at stream bit
// o + 128v - 1 (E[0] stands for stream bit -64..-1).  E (ew + 3 words), X and
// H must be zero and visible on entry.
template <uint32_t GROUP, uint32_t BATCH>
__device__ __forceinline__ void encode_windows(const uint64_t* src, uint32_t mw, const Layout& Lo, uint64_t* E,
                                               uint64_t* X, uint32_t* H, uint32_t gl)
{
    const uint32_t wins = Lo.windows(), last = mw - 1u;
    WindowWalk walk(Lo, gl);
    uint32_t ci = 0;
    uint64_t xacc = 0;
    uint32_t hacc = 0;
    for (uint32_t g0 = gl; g0 < wins; g0 += BATCH * GROUP) {
        uint64_t a[BATCH], b[BATCH], c[BATCH];
        uint32_t qm[BATCH], seg[BATCH], wd[BATCH], sh[BATCH], nn[BATCH], oo[BATCH], pp[BATCH];
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            walk.settle(Lo);
            uint32_t pw;
            const uint32_t m0 = walk.K + run_start(walk.v, pw);
            qm[u] = m0 >> 6;
            sh[u] = m0 & 63u;
            pp[u] = pw;
            seg[u] = walk.i;
            wd[u] = walk.v;
            nn[u] = walk.n;
            oo[u] = walk.o;
            walk.v += GROUP;
        }
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            a[u] = src[min(qm[u], last)];
            b[u] = src[min(qm[u] + 1u, last)];
            c[u] = src[min(qm[u] + 2u, last)];
        }
#pragma unroll
        for (uint32_t u = 0; u < BATCH; ++u) {
            if (g0 + u * GROUP >= wins) break;
            const uint32_t v = wd[u], pw = pp[u];
            uint64_t m0, m1;
            funnel128(a[u], b[u], c[u], sh[u], m0, m1);
            uint64_t x0, x1;
            if (v == 0) {
                x0 = head_expand(m0);
                x1 = ((m0 >> 57) | (m1 << 7)) << 1;        // positions 65..127
            } else {
                x0 = m0 << pw;
                x1 = (m1 << pw) | ((m0 >> 63) & pw);
            }
            mask_top(x0, x1, nn[u] - 128u * v);

            if (seg[u] != ci) {
                flush_partial(X, H, ci, xacc, hacc);
                ci = seg[u];
                xacc = 0;
                hacc = 0;
            }
            fold_window(x0, x1, v, xacc, hacc);

            const uint32_t sp = oo[u] + 128u * v + 63u;     // stream bit of position 128v, plus 64
            or128(E, sp >> 6, sp & 63u, x0, x1);
        }
    }
    flush_partial(X, H, ci, xacc, hacc);
    group_sync<GROUP>();
}

struct SegArgs {
    const uint64_t* enc;       // encoded arena (decode input, encode output)
    uint64_t enc_words;
    const hamming_seg_packet* descs;
    uint32_t n_packets;
    uint32_t max_msg_bytes;
    uint64_t* msg;             // message arena (decode output, encode input)
    uint64_t msg_words;
    uint16_t* syndromes;
    uint64_t syndrome_count;
    uint8_t* status;
    uint32_t slice_words;      // per-packet LDS buffer of the window form (accumulators excluded)
    uint32_t slot_dwords;      // LDS dwords per packet of the part form's kernels
    uint32_t run_words;        // words of the longest run that a wave of them can stage
    uint32_t cached;           // read packets with ordinary (1) or nontemporal (0) loads
};

// Per-packet accumulators after the buffer: X, one 64-bit word per segment,
// then H, one 32-bit word per segment.
constexpr uint32_t kAccWords = HAMMING_SEG_MAX_T + HAMMING_SEG_MAX_T / 2;

// Decode packet pk, of descriptor d, with GROUP threads (gl = 0..GROUP-1); Mb
// is the packet's message buffer in LDS (at least mw + 3 words) and acc its
// accumulators.  With GROUP < 64 several packets share a wave, so pk, the descriptor and the
// layout are per-lane values and wave-wide ballots are masked to the group.
// Every thread of a group takes the same branches at the barriers.  The descriptor
// comes by value: by reference its fields were loaded where they are used, 13
// loads with a wait each instead of two (2048 packets of 2000 bytes 7.3 against
// 6.8 us).
template <uint32_t GROUP, uint32_t BATCH>
__device__ __forceinline__ void decode_packet(const SegArgs& a, hamming_seg_packet d, uint64_t pk, uint32_t gl,
                                              uint64_t* Mb, uint64_t* acc)
{
    const uint32_t M = d.msg_bytes, t = d.t;
    Layout Lo;
    const bool shape_ok = make_layout(M, t, a.max_msg_bytes, Lo);
    const uint64_t ew = (uint64_t(Lo.total) + 63) / 64, mw = (uint64_t(M) + 7) / 8;
    const bool ok = shape_ok && d.enc_word_off <= a.enc_words && ew <= a.enc_words - d.enc_word_off &&
                    d.msg_word_off <= a.msg_words && mw <= a.msg_words - d.msg_word_off &&
                    (!a.syndromes || (d.seg_off <= a.syndrome_count && t <= a.syndrome_count - d.seg_off));
    if (!ok) {
        if (a.status && gl == 0) a.status[pk] = HAMMING_SEG_INVALID;
        return;
    }
    uint64_t* X = acc;
    uint32_t* H = reinterpret_cast<uint32_t*>(acc + HAMMING_SEG_MAX_T);
    for (uint32_t w = 2 * gl; w < mw + 3; w += 2 * GROUP) {   // in pairs: the slice has mw + 4 words
        Mb[w] = 0;
        Mb[w + 1] = 0;
    }
    for (uint32_t i = gl; i < t; i += GROUP) {
        X[i] = 0;
        H[i] = 0;
    }
    group_sync<GROUP>();

    decode_windows<GROUP, BATCH>(a.enc + d.enc_word_off, uint32_t(ew), Lo, Mb, X, H, gl);

    // checksum owners: thread gl takes segments gl, gl + GROUP, ...; an error
    // at a message position flips that message bit, one at a checksum
    // position changes no message bit
    uint32_t st = 0;
    for (uint32_t i = gl; i < t; i += GROUP) {
        const uint32_t s = fold_syndrome(X[i], H[i]), n = Lo.n(i);
        if (s >= 1 && s <= n) {
            if (s & (s - 1u)) {
                const uint32_t bit = Lo.K(i) + s - (31u - __clz(s)) - 2u;
                atomicXor(reinterpret_cast<unsigned long long*>(&Mb[bit >> 6]), 1ull << (bit & 63));
            }
            st = max(st, 1u);
        } else if (s > n) {
            st = 2;
        }
        if (a.syndromes) a.syndromes[d.seg_off + i] = uint16_t(s);
    }
    uint64_t mask = ~uint64_t(0);
    if constexpr (GROUP < 64) mask = ((uint64_t(1) << GROUP) - 1) << ((threadIdx.x & 63u) & ~(GROUP - 1));
    if constexpr (GROUP > 64) {
        // t <= 32: every owner is in the first wave, whose ballot decides
        mask = (threadIdx.x < 64) ? mask : 0;
    }
    const uint64_t any2 = __ballot(st == 2) & mask, any1 = __ballot(st == 1) & mask;
    if (a.status && gl == 0) a.status[pk] = any2 ? 2 : (any1 ? 1 : 0);
    group_sync<GROUP>();

    // the message words in 16-byte stores (two words per thread and step)
    uint64_t* dst = a.msg + d.msg_word_off;
    const uint64_t pairs = mw / 2;
    for (uint32_t q = gl; q < pairs; q += GROUP) {
        const uint64_t w0 = Mb[2 * q], w1 = Mb[2 * q + 1];
        u32x4 v;
        v.x = uint32_t(w0);
        v.y = uint32_t(w0 >> 32);
        v.z = uint32_t(w1);
        v.w = uint32_t(w1 >> 32);
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4a8*>(dst) + q);
    }
    if ((mw & 1) && gl == 0) __builtin_nontemporal_store(Mb[mw - 1], dst + mw - 1);
}

// Encode a packet of descriptor d with GROUP threads; E is the packet's encoded
// buffer in LDS (at least ew + 3 words, E[0] in front of the stream) and acc its
// accumulators.  A descriptor this launch cannot take is skipped.
template <uint32_t GROUP, uint32_t BATCH>
__device__ __forceinline__ void encode_packet(const SegArgs& a, hamming_seg_packet d, uint32_t gl, uint64_t* E,
                                              uint64_t* acc)
{
    const uint32_t M = d.msg_bytes, t = d.t;
    Layout Lo;
    const bool shape_ok = make_layout(M, t, a.max_msg_bytes, Lo);
    const uint64_t ew = (uint64_t(Lo.total) + 63) / 64, mw = (uint64_t(M) + 7) / 8;
    const bool ok = shape_ok && d.enc_word_off <= a.enc_words && ew <= a.enc_words - d.enc_word_off &&
                    d.msg_word_off <= a.msg_words && mw <= a.msg_words - d.msg_word_off;
    if (!ok) return;
    uint64_t* X = acc;
    uint32_t* H = reinterpret_cast<uint32_t*>(acc + HAMMING_SEG_MAX_T);
    for (uint32_t w = gl; w < ew + 3; w += GROUP) E[w] = 0;
    for (uint32_t i = gl; i < t; i += GROUP) {
        X[i] = 0;
        H[i] = 0;
    }
    group_sync<GROUP>();

    encode_windows<GROUP, BATCH>(a.msg + d.msg_word_off, uint32_t(mw), Lo, E, X, H, gl);

    // checksum position 2^j of segment i takes bit j of the syndrome of its
    // message bits, which makes the segment's syndrome 0
    for (uint32_t i = gl; i < t; i += GROUP) {
        const uint32_t s = fold_syndrome(X[i], H[i]), o = Lo.o(i);
        for (uint32_t j = 0; (s >> j) != 0; ++j) {
            if (!((s >> j) & 1u)) continue;
            const uint32_t bit = o + (1u << j) + 63u;       // stream bit of position 2^j, plus 64
            atomicOr(reinterpret_cast<unsigned long long*>(&E[bit >> 6]), 1ull << (bit & 63));
        }
    }
    group_sync<GROUP>();

    // the encoded words in 16-byte stores (two words per thread and step)
    uint64_t* dst = const_cast<uint64_t*>(a.enc) + d.enc_word_off;
    const uint64_t pairs = ew / 2;
    for (uint32_t q = gl; q < pairs; q += GROUP) {
        const uint64_t w0 = E[2 * q + 1], w1 = E[2 * q + 2];
        u32x4 v;
        v.x = uint32_t(w0);
        v.y = uint32_t(w0 >> 32);
        v.z = uint32_t(w1);
        v.w = uint32_t(w1 >> 32);
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4a8*>(dst) + q);
    }
    if ((ew & 1) && gl == 0) __builtin_nontemporal_store(E[ew], dst + ew - 1);
}

// ---- part form ---------------------------------------------------------------
//
// The packets of a wave that lie end to end in both arenas, or have one shape
// and lie at one stride in either (a gap after each), take this form: their
// words are one run, which the 64 lanes copy into LDS and the results out of it
// in whole cache lines.  The bits are then dealt by segment: every lane owns
// one part of one segment (seg_parts.h), reads it from LDS into registers,
// folds its syndrome there and ORs its message (or encoded) bits into place
// over the run it came from.
//
// What bounded the window form was neither its instructions nor its latency
// but how its loads met the memory: a group's loads start wherever its packet
// does and cover 128 or 256 bytes, so most cache lines were asked for twice.
// A copy of the kernel with all bit work taken out ran no faster (1200-byte
// packets, t = 4, 2^19 of them: 253-285 us, decoding 256-281 us); moving the
// same words as one run per wave, with the bit work, takes 200 us (6.4 TB/s).
// Encoding 2^18 packets of 800 bytes, t = 5: 104 -> 75 us (5.7 TB/s).  Packets of
// several shapes hold their layout per lane instead of per wave, and a lane
// waits for the longest part: 2^18 of 400 to 2000 bytes, t = 2 to 6, decode
// 181 -> 141 us, encode 204 -> 148; of 400 to 800 bytes 98 -> 88, 106 -> 77.

typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr uint32_t kPartLoads = 8;          // 16-byte loads a lane has in flight while a run is staged
constexpr uint32_t kPartStores = 4;         // 16-byte vectors it reads back before it stores the first
constexpr uint32_t kPartPad = 4;            // dwords in front of the run

// The wave's LDS: the run's area (the pad, the run's shift within a line, the run,
// what is cleared and ORed in after it) in blocks, then one syndrome per lane, then
// kPartSlack dwords.  Lanes past their segment's last window read up to 39 + 4 NW
// dwords past the pad and the run's words, which the syndromes and the slack cover.
constexpr uint32_t kPartEnds = kPartPad + 30u + 8u;
constexpr uint32_t kPartSlack = 12u;

// LDS dword of area dword a; BLOCKS: the area lies in blocks (seg_parts.h).
template <bool BLOCKS>
__device__ __forceinline__ uint32_t place(uint32_t a)
{
    return BLOCKS ? block_at(a) : a;
}

// A run of consecutive 64-bit words that a wave moves between global memory
// and LDS in 16-byte vectors, lane 0 starting on a 128-byte line: word w of
// the run is dword kPartPad + 2 (shift + w) of its area,
// vector j holds words 2j - shift and 2j + 1 - shift, and vectors lo .. hi - 1 lie in the run
// altogether.  The first and the last word may lie in no whole vector; they
// are moved alone, so no access leaves the run.
template <bool BLOCKS>
struct Run {
    uint32_t words, shift, lo, hi;

    __device__ Run(const void* first_word, uint32_t words_)
        : words(words_), shift(uint32_t(reinterpret_cast<uintptr_t>(first_word) >> 3) & 15u),
          lo((shift + 1u) / 2u), hi((shift + words) / 2u) {}

    // Area dword of word w, and LDS place of vector j.
    __device__ uint32_t at(uint32_t w) const { return kPartPad + 2u * (shift + w); }

    static __device__ u32x4* vector(uint32_t* S, uint32_t j)
    {
        return reinterpret_cast<u32x4*>(S + place<BLOCKS>(kPartPad + 4u * j));
    }
    static __device__ const u32x4* vector(const uint32_t* S, uint32_t j)
    {
        return reinterpret_cast<const u32x4*>(S + place<BLOCKS>(kPartPad + 4u * j));
    }

    template <bool NT>
    __device__ __forceinline__ void load(const uint64_t* src, uint32_t* S, uint32_t lane) const
    {
        const char* from = reinterpret_cast<const char*>(src - shift);     // uniform: loads take a 32-bit offset
        const uint32_t edge = lane == 0 ? 0u : words - 1u;
        uint64_t edge_word = 0;
        if (lane < 2) edge_word = src[edge];
        for (uint32_t base = 0; base < hi && lo < hi; base += kPartLoads * 64) {
            u32x4 x[kPartLoads];
            uint32_t j[kPartLoads];
            // lanes outside the run move its first or last whole vector once
            // more: a load under a branch of its own would wait for the others
#pragma unroll
            for (uint32_t u = 0; u < kPartLoads; ++u) {
                if (base + u * 64 >= hi) continue;
                j[u] = min(max(base + u * 64 + lane, lo), hi - 1u);
                const u32x4a8* v = reinterpret_cast<const u32x4a8*>(from + 16u * j[u]);
                x[u] = NT ? __builtin_nontemporal_load(v) : *v;
            }
#pragma unroll
            for (uint32_t u = 0; u < kPartLoads; ++u)
                if (base + u * 64 < hi) {
                    u32x4* const to = vector(S, j[u]);
                    *to = x[u];
                    if (BLOCKS && (kPartPad / 4u + j[u]) % (kBlockDwords / 4u) == 0) to[-1] = x[u];
                }
        }
        if (lane < 2) {
            uint2* const to = reinterpret_cast<uint2*>(S + place<BLOCKS>(at(edge)));
            const uint2 y = make_uint2(uint32_t(edge_word), uint32_t(edge_word >> 32));
            *to = y;
            if (BLOCKS && at(edge) % kBlockDwords < kBlockRoom) to[-int(kBlockRoom / 2)] = y;
        }
    }

    // Clears the run's dwords in LDS and at least `more` dwords after them, the
    // blocks' rooms included.
    __device__ __forceinline__ void clear(uint32_t more, uint32_t* S, uint32_t lane) const
    {
        const uint32_t last = place<BLOCKS>(kPartPad + 2u * (shift + words) + more - 1u);
        for (uint32_t j = kPartPad / 4u + lane; 4u * j <= last; j += 64)
            reinterpret_cast<u32x4*>(S)[j] = u32x4{0u, 0u, 0u, 0u};
    }

    // Blocks only: merges the rooms into the blocks after them.  Others may set or flip bits of
    // the run at the same time: no two of these touch one bit.
    __device__ __forceinline__ void merge(uint32_t* S, uint32_t lane) const
    {
        if constexpr (!BLOCKS) return;
        constexpr uint32_t STEP = kBlockDwords + kBlockRoom;
        for (uint32_t b = lane + 1u; b * kBlockDwords < kPartPad + 2u * (shift + words); b += 64) {
            const u32x4 x = *reinterpret_cast<const u32x4*>(S + b * STEP - kBlockRoom);
#pragma unroll
            for (int k = 0; k < 4; ++k) atomicXor(S + b * STEP + k, x[k]);
        }
    }

    // Stores the run.  Of every `stride` words of it `packet` are a packet's and
    // the rest the gap after it, which is left as it was.
    __device__ __forceinline__ void store(uint64_t* dst, const uint32_t* S, uint32_t lane, uint32_t packet,
                                          uint32_t stride) const
    {
        if (packet != stride) {
            for (uint32_t j = lane; j < (shift + words + 1u) / 2u; j += 64) {
                const u32x4 x = *vector(S, j);
                const int32_t w = int32_t(2u * j) - int32_t(shift);                  // the vector's first word
                const uint32_t in0 = w < 0 ? packet : uint32_t(w) - small_div(uint32_t(w), stride) * stride;
                const uint32_t in1 = w + 1 < 0 ? packet : w < 0 || in0 + 1u == stride ? 0u : in0 + 1u;
                const bool has0 = in0 < packet, has1 = in1 < packet && uint32_t(w + 1) < words;
                if (has0 && has1)
                    __builtin_nontemporal_store(x, reinterpret_cast<u32x4a8*>(dst + w));
                else if (has0)
                    __builtin_nontemporal_store(uint64_t(x.x) | (uint64_t(x.y) << 32), dst + w);
                else if (has1)
                    __builtin_nontemporal_store(uint64_t(x.z) | (uint64_t(x.w) << 32), dst + w + 1);
            }
            return;
        }
        char* to = reinterpret_cast<char*>(dst - shift);
        for (uint32_t base = 0; base < hi; base += kPartStores * 64) {
            u32x4 x[kPartStores];
#pragma unroll
            for (uint32_t u = 0; u < kPartStores; ++u) {
                if (base + u * 64 >= hi) continue;
                x[u] = *vector(S, min(base + u * 64 + lane, hi - 1u));
            }
#pragma unroll
            for (uint32_t u = 0; u < kPartStores; ++u) {
                const uint32_t j = base + u * 64 + lane;
                if (j >= lo && j < hi) __builtin_nontemporal_store(x[u], reinterpret_cast<u32x4a8*>(to + 16u * j));
            }
        }
        if (lane < 2 && ((lane == 0 ? shift : shift + words) & 1u)) {
            const uint32_t w = lane == 0 ? 0u : words - 1u;
            const uint2 y = *reinterpret_cast<const uint2*>(S + place<BLOCKS>(at(w)));
            __builtin_nontemporal_store(uint64_t(y.x) | (uint64_t(y.y) << 32), dst + w);
        }
    }
};

__device__ __forceinline__ uint64_t readfirstlane64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    return lo | (uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32))) << 32);
}

// A lane's part: windows v0 .. v0 + cnt - 1 of segment i (none when cnt = 0).
struct Part {
    uint32_t i, v0, cnt, K, o;
    int32_t n;

    __device__ Part(const Layout& Lo, const hm::Parts& P, uint32_t gl)
    {
        const uint32_t seg = P.segment(gl);
        const bool mine = seg < Lo.t;
        i = mine ? seg : 0u;
        v0 = (gl - seg * P.parts) * P.len;
        K = Lo.K(i);
        o = Lo.o(i);
        n = mine ? int32_t(Lo.n(i)) : -1;
        const uint32_t nv = mine ? (i < Lo.rem ? Lo.vA : Lo.vB) : 0u;
        v0 = min(v0, nv);
        cnt = min(nv - v0, P.len);
    }
};

// Window of five dwords from area dword a, bit sh (mod 32), on: four dwords.
template <bool BLOCKS>
__device__ __forceinline__ void read_window(const uint32_t* S, uint32_t a, uint32_t sh, uint32_t (&x)[4])
{
    const uint32_t* p = S + place<BLOCKS>(a);
    const u32x4 w = *reinterpret_cast<const u32x4a4*>(p);
    const uint32_t e = p[4];
    x[0] = hm::align32(w.y, w.x, sh);
    x[1] = hm::align32(w.z, w.y, sh);
    x[2] = hm::align32(w.w, w.z, sh);
    x[3] = hm::align32(e, w.w, sh);
}

// ORs a placed window in, its dword 0 being area dword a.
template <bool BLOCKS>
__device__ __forceinline__ void or_window(uint32_t* S, uint32_t a, const hm::Placed& w)
{
    uint32_t* p = S + place<BLOCKS>(a + uint32_t(w.first));
#pragma unroll
    for (int k = 0; k < 5; ++k) atomicOr(p + k, w.y[k]);
}

// The packets of a wave: this lane's packet's layout, parts and first word in
// either run (e0, m0), the most windows of a part (len), the words of the runs
// and their first words, and for packets with gaps between them (packet !=
// stride) the words of one and from one to the next.  W is the wave's LDS and
// X (within it) one syndrome per lane.
struct WaveRun {
    Layout Lo;
    hm::Parts P;
    uint32_t e0, m0, len, eruns, mruns;
    uint32_t ew, mw, es, ms;
    uint64_t *enc, *msg;
    uint32_t *W, *X;
};

// Whether equal packets lie so that about half of their parts or more begin in the
// banks of the first one, in either run: segments, parts and packets a multiple of
// 16 dwords (512 bits) apart, all of them.  Lanes step through their parts together,
// so such lanes wait for each other at every access, and the wave stages its runs
// in blocks instead.  2^18 packets, decode and encode: 633 bytes, t = 5 (every lane
// in one bank) 151 and 156 -> 73 and 75 us; 2^17: 1908 bytes, t = 5 193 and 202 -> 88
// and 87, 1020 bytes, t = 2 (half of the lanes) 81 and 82 -> 45 and 48, 384 bytes,
// t = 2 27 and 26 -> 22 and 24.  Blocks cost an address per window, a second store
// per block and the merge, so other shapes do without: they would take 3-15% longer,
// and steps of 28 dwords would meet in one bank (1600 bytes, t = 2 73 against 133
// us).  In scalar instructions, most waves leaving after the first two: counting
// the lanes with ballots cost every other shape 1-4%.
__device__ __forceinline__ bool lanes_collide(const WaveRun& r)
{
    // t - 1 steps of `bits` stay within the 3 dwords before or after a multiple of m
    const auto near = [&](uint32_t bits, uint32_t m) {
        const int32_t d = int32_t((bits + m / 2u) % m) - int32_t(m / 2u);
        return uint32_t(d < 0 ? -d : d) * (r.Lo.t - 1u) <= 112u;
    };
    const auto side = [&](uint32_t words, uint32_t bits) {
        if (words % 8u) return false;
        if (r.P.parts == 1 || r.len % 4u == 0) return near(bits, 512u);
        return r.P.parts == 2 && words % 16u == 0 && near(bits, 1024u);
    };
    return side(r.es, r.Lo.nA) || side(r.ms, r.Lo.q);
}

// Decodes the wave's packets with GROUP lanes each, every lane its part.  The
// messages are built over the received words once every lane holds its
// windows in registers.
template <uint32_t GROUP, uint32_t NW, bool BLOCKS>
__device__ __forceinline__ void decode_parts(const SegArgs& a, const WaveRun& r, uint64_t pk, uint64_t seg_off)
{
    const uint32_t lane = threadIdx.x & 63u, gl = lane % GROUP, slot = lane / GROUP;
    const Layout& Lo = r.Lo;
    const hm::Parts& P = r.P;
    uint32_t* S = r.W;
    uint32_t* X = r.X + slot * GROUP;
    const Run<BLOCKS> in(r.enc, r.eruns), out(r.msg, r.mruns);
    const uint32_t mb = out.at(r.m0);
    X[gl] = 0;
    if (a.cached)
        in.template load<false>(r.enc, S, lane);
    else
        in.template load<true>(r.enc, S, lane);
    wave_sync();

    const Part pt(Lo, P, gl);
    const uint32_t bit = pt.o + 128u * pt.v0 + 32u * in.at(r.e0) - 1u;   // area bit of position 128 v0
    const int32_t last = min(pt.n, int32_t(128u * (pt.v0 + P.len)) - 1);        // the part's last position
    hm::PartSyndrome syn;
    uint32_t x[NW][4];
#pragma unroll
    for (uint32_t u = 0; u < NW; ++u) {
        if (u < r.len) {
            read_window<BLOCKS>(S, (bit >> 5) + 4u * u, bit, x[u]);
            const int32_t top = last - int32_t(128u * (pt.v0 + u));
            if (top < 127) hm::mask_window(x[u], top);
            if (u == 0) x[0][0] &= pt.v0 == 0 ? ~1u : ~0u;              // there is no position 0
            syn.add(x[u], pt.v0 + u);
        }
    }
    const uint32_t sv = syn.value();
    if (sv) atomicXor(&X[pt.i], sv);
    wave_sync();
    out.clear(5u, S, lane);
    wave_sync();
    // v0 anew: v0 + u would be held for every window from the first loop on
    uint32_t v0 = pt.v0;
    asm volatile("" : "+v"(v0));
#pragma unroll
    for (uint32_t u = 0; u < NW; ++u) {
        if (u < pt.cnt) {
            const uint32_t v = v0 + u;
            uint32_t at = pt.K + hm::run_base(v);
            if (u == 0 && v == 0) {
                hm::compact_head(x[0]);
                at = pt.K;
            } else {
                x[u][0] &= ~hm::is_pow2_window(v);
            }
            or_window<BLOCKS>(S, mb, hm::place_window(x[u], at));
        }
    }
    wave_sync();

    // checksum owners: lane gl has segment gl; an error at a message position
    // flips that message bit, one at a checksum position changes none
    out.merge(S, lane);
    uint32_t st = 0;
    if (gl < Lo.t) {
        const uint32_t s = X[gl], n = Lo.n(gl);
        if (s >= 1 && s <= n) {
            if (s & (s - 1u)) {
                const uint32_t b = Lo.K(gl) + s - (31u - __clz(s)) - 2u;
                atomicXor(&S[place<BLOCKS>(mb + (b >> 5))], 1u << (b & 31u));
            }
            st = 1;
        } else if (s > n) {
            st = 2;
        }
        if (a.syndromes) a.syndromes[seg_off + gl] = uint16_t(s);
    }
    uint64_t mask = ~uint64_t(0);
    if constexpr (GROUP < 64) mask = ((uint64_t(1) << GROUP) - 1) << (slot * GROUP);
    const uint64_t any2 = __ballot(st == 2) & mask, any1 = __ballot(st == 1) & mask;
    if (a.status && gl == 0) a.status[pk] = any2 ? 2 : (any1 ? 1 : 0);
    wave_sync();
    out.store(r.msg, S, lane, r.mw, r.ms);
}

// Encodes the wave's packets: the same parts, each window built from its run
// of message bits and placed into the encoded packet.
template <uint32_t GROUP, uint32_t NW, bool BLOCKS>
__device__ __forceinline__ void encode_parts(const SegArgs& a, const WaveRun& r)
{
    const uint32_t lane = threadIdx.x & 63u, gl = lane % GROUP, slot = lane / GROUP;
    const Layout& Lo = r.Lo;
    const hm::Parts& P = r.P;
    uint32_t* S = r.W;
    uint32_t* X = r.X + slot * GROUP;
    const Run<BLOCKS> in(r.msg, r.mruns), out(r.enc, r.eruns);
    const uint32_t mb = in.at(r.m0), eb = out.at(r.e0);
    X[gl] = 0;
    if (a.cached)
        in.template load<false>(r.msg, S, lane);
    else
        in.template load<true>(r.msg, S, lane);
    wave_sync();

    const Part pt(Lo, P, gl);
    hm::PartSyndrome syn;
    uint32_t x[NW][4];
#pragma unroll
    for (uint32_t u = 0; u < NW; ++u) {
        if (u < pt.cnt) {
            const uint32_t v = pt.v0 + u;
            const bool head = u == 0 && v == 0;
            const uint32_t at = pt.K + (head ? 0u : hm::run_base(v));
            read_window<BLOCKS>(S, mb + (at >> 5), at, x[u]);
            if (head)
                hm::expand_head(x[u]);
            else
                x[u][0] &= ~hm::is_pow2_window(v);
            const int32_t top = pt.n - int32_t(128u * v);
            if (top < 127) hm::mask_window(x[u], top);
            syn.add(x[u], v);
        }
    }
    const uint32_t sv = syn.value();
    if (sv) atomicXor(&X[pt.i], sv);
    wave_sync();
    out.clear(6u, S, lane);
    wave_sync();
#pragma unroll
    for (uint32_t u = 0; u < NW; ++u) {
        // one dword further on, so that the stream bit is never negative
        if (u < pt.cnt) or_window<BLOCKS>(S, eb - 1u, hm::place_window(x[u], pt.o + 128u * (pt.v0 + u) + 31u));
    }
    wave_sync();

    // checksum position 2^j of segment gl takes bit j of the syndrome of its
    // message bits, which makes the segment's syndrome 0
    out.merge(S, lane);
    if (gl < Lo.t) {
        const uint32_t s = X[gl], o = Lo.o(gl);
        const uint32_t w = (s & 3u) | ((s & 4u) << 1) | ((s & 8u) << 4) | ((s & 16u) << 11) | ((s & 32u) << 26);
        atomicOr(&S[place<BLOCKS>(eb + (o >> 5))], w << (o & 31u));
        atomicOr(&S[place<BLOCKS>(eb + (o >> 5) + 1u)], (w >> 1) >> (31u - (o & 31u)));
        for (uint32_t j = 6; (s >> j) != 0; ++j) {
            const uint32_t b = o + (1u << j) - 1u;
            if ((s >> j) & 1u) atomicOr(&S[place<BLOCKS>(eb + (b >> 5))], 1u << (b & 31u));
        }
    }
    wave_sync();
    out.store(r.enc, S, lane, r.ew, r.es);
}

// Consecutive blocks that each XCD takes in turn (xcd_block): the lines that two
// blocks share then meet in one L2.  2000-byte packets 353 against 362 us
// without, 400 to 1200 bytes within 1-3% either way.
constexpr uint32_t kSegXcdChunk = 8;

// Shortest message of the part form, whose fixed work outweighs its loads below:
// 128-byte packets 30.2 against 28.6 us in the window form, 250-byte ones 33
// against 48.
constexpr uint32_t kPartMinBytes = 192;

// 256 / GROUP packets per block, GROUP <= 64 lanes each.  A wave takes the part
// form when all its packets are there, have at least kPartMinBytes and parts
// that fit NW windows, and lie end to end in both arenas or, being of one
// shape, at one stride in either, their runs inside the arenas and inside the
// wave's LDS; the window form otherwise.  NW = 8 fits the 72 registers that let
// 7 waves share a SIMD; without the bound the compiler takes 78 (800-byte
// packets 166 against 160 us).
template <uint32_t GROUP, uint32_t NW, uint32_t BATCH, bool DECODE>
__global__ __launch_bounds__(64 * kSegWaves) __attribute__((amdgpu_waves_per_eu(NW == 8 ? 7 : 1)))
void seg_parts_kernel(SegArgs a)
{
    constexpr uint32_t PACKETS = 64 / GROUP;                     // of a wave
    extern __shared__ uint64_t lds[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
    const uint32_t lane = threadIdx.x & 63u, gl = lane % GROUP, slot = lane / GROUP;
    const uint64_t pk = (uint64_t(hm::xcd_block(blockIdx.x, gridDim.x, kSegXcdChunk)) * kSegWaves + wave) * PACKETS + slot;
    if (pk >= a.n_packets) return;
    WaveRun r;
    const uint32_t wave_dwords = PACKETS * a.slot_dwords;
    r.W = reinterpret_cast<uint32_t*>(lds) + wave * wave_dwords;
    r.X = r.W + wave_dwords - kPartSlack - 64u;
    const hamming_seg_packet d = a.descs[pk];
    const uint32_t M = __builtin_amdgcn_readfirstlane(d.msg_bytes), t = __builtin_amdgcn_readfirstlane(d.t);
    // all 64 lanes are there, and their packets have one shape
    const bool one_shape = __ballot(d.msg_bytes == M && d.t == t) == ~uint64_t(0);
    if (one_shape && t <= GROUP && (GROUP == 64 || M >= kPartMinBytes) && make_layout(M, t, a.max_msg_bytes, r.Lo)) {
        const uint64_t e0 = readfirstlane64(d.enc_word_off), m0 = readfirstlane64(d.msg_word_off);
        r.P = hm::make_parts(t, r.Lo.rem ? r.Lo.vA : r.Lo.vB, GROUP);
        r.ew = (r.Lo.total + 63u) / 64u;
        r.mw = (M + 7u) / 8u;
        r.es = r.ew;
        r.ms = r.mw;
        if constexpr (PACKETS > 1) {
            r.es = __builtin_amdgcn_readlane(uint32_t(d.enc_word_off - e0), GROUP);        // packet 1's distance
            r.ms = __builtin_amdgcn_readlane(uint32_t(d.msg_word_off - m0), GROUP);
        }
        bool alike = d.enc_word_off == e0 + uint64_t(slot) * r.es && d.msg_word_off == m0 + uint64_t(slot) * r.ms;
        if constexpr (DECODE)
            alike = alike && (!a.syndromes || (d.seg_off <= a.syndrome_count && t <= a.syndrome_count - d.seg_off));
        const uint32_t most = a.run_words;
        const bool apart = r.es >= r.ew && r.ms >= r.mw && r.es <= most && r.ms <= most;
        r.eruns = (PACKETS - 1) * r.es + r.ew;
        r.mruns = (PACKETS - 1) * r.ms + r.mw;
        if (r.P.len <= NW && apart && r.eruns <= most && r.mruns <= most && e0 <= a.enc_words &&
            r.eruns <= a.enc_words - e0 && m0 <= a.msg_words && r.mruns <= a.msg_words - m0 &&
            __ballot(alike) == ~uint64_t(0)) {
            r.enc = const_cast<uint64_t*>(a.enc) + e0;
            r.msg = a.msg + m0;
            r.e0 = slot * r.es;
            r.m0 = slot * r.ms;
            r.len = r.P.len;
            if (PACKETS > 1 && lanes_collide(r)) {
                if constexpr (DECODE)
                    decode_parts<GROUP, NW, PACKETS != 1>(a, r, pk, d.seg_off);
                else
                    encode_parts<GROUP, NW, PACKETS != 1>(a, r);
                return;
            }
            if constexpr (DECODE)
                decode_parts<GROUP, NW, false>(a, r, pk, d.seg_off);
            else
                encode_parts<GROUP, NW, false>(a, r);
            return;
        }
    }
    if (PACKETS > 1 && !one_shape) {
        // packets of several shapes, end to end.  What tells without a layout that
        // they are not comes first: with gaps between them the wave takes the window
        // form, and the layout in front of that cost it 10% (2^18 packets of 400 to
        // 2000 bytes 189 us, 177 now, 171 in a kernel of the window form alone)
        const uint32_t most = a.run_words;
        const uint32_t mw = (d.msg_bytes + 7u) / 8u, first = uint32_t(d.msg_word_off);
        const uint32_t before = __shfl_up(first + mw, GROUP);                          // the packet before ends here
        bool ok = d.t <= GROUP && d.msg_bytes >= kPartMinBytes && (slot == 0 || first == before);
        if constexpr (DECODE)
            ok = ok && (!a.syndromes || (d.seg_off <= a.syndrome_count && d.t <= a.syndrome_count - d.seg_off));
        if (__ballot(ok) == ~uint64_t(0) &&
            __ballot(make_layout(d.msg_bytes, d.t, a.max_msg_bytes, r.Lo)) == ~uint64_t(0)) {
            const uint64_t e0 = readfirstlane64(d.enc_word_off), m0 = readfirstlane64(d.msg_word_off);
            r.P = hm::make_parts(d.t, r.Lo.rem ? r.Lo.vA : r.Lo.vB, GROUP);
            const uint32_t ew = (r.Lo.total + 63u) / 64u;
            r.eruns = r.mruns = r.len = 0;
#pragma unroll
            for (uint32_t k = 0; k < PACKETS; ++k) {
                if (slot == k) {
                    r.e0 = r.eruns;
                    r.m0 = r.mruns;
                }
                r.eruns += __builtin_amdgcn_readlane(ew, k * GROUP);
                r.mruns += __builtin_amdgcn_readlane(mw, k * GROUP);
                r.len = max(r.len, uint32_t(__builtin_amdgcn_readlane(r.P.len, k * GROUP)));
            }
            const bool in_line = d.enc_word_off == e0 + r.e0 && d.msg_word_off == m0 + r.m0;
            if (r.len <= NW && r.eruns <= most && r.mruns <= most && e0 <= a.enc_words &&
                r.eruns <= a.enc_words - e0 && m0 <= a.msg_words && r.mruns <= a.msg_words - m0 &&
                __ballot(in_line) == ~uint64_t(0)) {
                r.enc = const_cast<uint64_t*>(a.enc) + e0;
                r.msg = a.msg + m0;
                r.ew = r.es = r.mw = r.ms = 0;
                if constexpr (DECODE)
                    decode_parts<GROUP, NW, false>(a, r, pk, d.seg_off);
                else
                    encode_parts<GROUP, NW, false>(a, r);
                return;
            }
        }
    }
    if constexpr (GROUP == 64) {
        // one packet of any valid shape fits its wave, so this one is not valid
        if constexpr (DECODE)
            if (a.status && gl == 0) a.status[pk] = HAMMING_SEG_INVALID;
    } else {
        uint64_t* slice = reinterpret_cast<uint64_t*>(r.W + slot * a.slot_dwords);
        if constexpr (DECODE)
            decode_packet<GROUP, BATCH>(a, d, pk, gl, slice, slice + a.slice_words);
        else
            encode_packet<GROUP, BATCH>(a, d, gl, slice, slice + a.slice_words);
    }
}

// The window form alone, 256 / GROUP packets per block: a workgroup per packet, the
// latency form, and batches of packets too short for the part form, which would
// only pay for its checks (2^18 packets of 128 bytes 31.7 against 30.5 us).  The
// packet is a per-lane value for every GROUP: from blockIdx alone a workgroup's one
// descriptor and its layout would go through the scalar unit, which takes longer
// (1500 packets with gaps 6.45 against 6.2 us).
template <uint32_t GROUP, uint32_t BATCH>
__global__ __launch_bounds__(64 * kSegWaves) void seg_decode_kernel(SegArgs a)
{
    extern __shared__ uint64_t lds[];
    const uint32_t slot = threadIdx.x / GROUP;
    const uint64_t pk = uint64_t(blockIdx.x) * (64 * kSegWaves / GROUP) + slot;
    if (pk >= a.n_packets) return;
    uint64_t* slice = lds + slot * (a.slice_words + kAccWords);
    decode_packet<GROUP, BATCH>(a, a.descs[pk], pk, threadIdx.x % GROUP, slice, slice + a.slice_words);
}

template <uint32_t GROUP, uint32_t BATCH>
__global__ __launch_bounds__(64 * kSegWaves) void seg_encode_kernel(SegArgs a)
{
    extern __shared__ uint64_t lds[];
    const uint32_t slot = threadIdx.x / GROUP;
    const uint64_t pk = uint64_t(blockIdx.x) * (64 * kSegWaves / GROUP) + slot;
    if (pk >= a.n_packets) return;
    uint64_t* slice = lds + slot * (a.slice_words + kAccWords);
    encode_packet<GROUP, BATCH>(a, a.descs[pk], threadIdx.x % GROUP, slice, slice + a.slice_words);
}

// Threads per packet when the caller leaves the choice to the library: a
// workgroup per packet for batches too small to fill the GPU's wave slots
// (latency), otherwise a group sized to the packets (throughput).
constexpr uint32_t kWideMaxPackets = 2048;
std::atomic<uint32_t> g_seg_threads{0};

uint32_t auto_threads_per_packet(uint32_t n_packets, uint32_t max_msg_bytes)
{
    if (n_packets <= kWideMaxPackets) return 256;
    // 8 lanes share the per-packet work between eight packets of a wave, 16 have
    // fewer windows each.  Up to 633 bytes 8 are faster (from 16384 packets on; 2^17
    // equal packets of 560 bytes, 16 against 8, mean of t = 2 to 6: decode 1.16 times
    // as long, encode 1.09; 633 bytes 1.07 and 1.08), from 634 on, where parts of t = 5
    // have nine windows on 8 lanes, 16 (640 bytes 0.96 and 0.99, 700 bytes 0.91 and 0.93;
    // 2100 packets of 640 bytes 0.79 and 0.78; slower only at 32768 packets, encoding,
    // by 2-9%).  They win up to 2000 bytes (2^19 packets 339 us, 32: 344) for every t
    if (max_msg_bytes <= 633u) return 8u;
    // Up to 4096 packets 16 lanes each leave a SIMD one wave, 32 two.  Decode
    // and encode, 32 against 16: 4096 equal packets of 2000 bytes 6.8 and 7.0
    // against 7.9 and 7.7 us, 400..2000 bytes 7.3 and 8.1 against 8.4 and 9.4;
    // at 1200 bytes (5.9 and 6.2) and with 6000 packets no difference.
    if (n_packets <= 4096 && max_msg_bytes > 1000 && max_msg_bytes <= 2048) return 32u;
    return max_msg_bytes <= 2048 ? 16u : (max_msg_bytes <= 3072 ? 32u : 64u);
}

// LDS dwords per packet of the part form's kernels (a wave has 64 / group): its
// share of a wave whose packets are the largest (at most 16 checksum bits for each
// of t <= group segments); at least what the window form takes.
uint32_t part_slot_dwords(uint32_t max_msg_bytes, uint32_t group, uint32_t slice_words)
{
    const uint32_t ew = (8u * max_msg_bytes + 16u * (group < HAMMING_SEG_MAX_T ? group : HAMMING_SEG_MAX_T) + 63u) / 64u;
    const uint32_t packets = 64u / group;
    // block_capacity may lose up to four dwords of an area to its rounding
    const uint32_t wave = block_area(2u * packets * ew + kPartEnds + 4u) + 64u + kPartSlack;
    const uint32_t parts = (wave + packets - 1u) / packets;
    const uint32_t windows = group < 64 ? 2u * (slice_words + kAccWords) : 0u;
    return ((parts > windows ? parts : windows) + 3u) & ~3u;
}

// The kernel for GROUP lanes per packet, with registers for 8 (encoding 9: the
// compiler then needs 65 registers, with 8 it takes 86), 12 or 15 windows in a lane.
// A lane's share is max_msg_bytes / (16 GROUP) windows if all lanes have one; the
// largest share of t <= 8 segments is about 1.5 times that.  Where the caller sets 8
// lanes, t = 5 has nine windows from 634 bytes on (2^18 packets of 634 bytes, decode 76
// us, 86 in the window form).  On 16 lanes t = 9 and 10 have more than 12 from
// 1715 bytes on (2000 bytes, t = 10, decode 253 us in the window form, 180 with 15
// windows, t = 9 229 and 180; t <= 6 0-1% slower than with 12).
// The window form loads 2 windows ahead while a thread has about five of them
// (unused slots of a last batch cost loads and walk steps), 4 above (more
// loads in flight); measured on the Table 1 grid.
template <uint32_t GROUP, bool DECODE>
void (*part_kernel(uint32_t max_msg_bytes))(SegArgs)
{
    if constexpr (GROUP == 64) {
        return seg_parts_kernel<64, 6, 2, DECODE>;       // six are enough for every shape
    } else {
        const bool wide = max_msg_bytes > (GROUP == 8 && DECODE ? 633u : 80u * GROUP);
        if constexpr (GROUP == 16)
            if (max_msg_bytes > 1714u) return seg_parts_kernel<GROUP, 15, 4, DECODE>;
        return wide ? seg_parts_kernel<GROUP, 12, 4, DECODE> : seg_parts_kernel<GROUP, DECODE ? 8 : 9, 2, DECODE>;
    }
}

// The window form's kernel for GROUP threads per packet; two windows ahead, as short
// packets and a workgroup's share have few.
template <uint32_t GROUP, bool DECODE>
constexpr void (*window_kernel())(SegArgs)
{
    if constexpr (DECODE)
        return seg_decode_kernel<GROUP, 2>;
    else
        return seg_encode_kernel<GROUP, 2>;
}

// Batches of at most this many message bytes are read with ordinary loads,
// larger ones with nontemporal loads; half the 256 MB Infinity Cache can still
// hold them.  Decoding, ordinary against nontemporal loads by where the batch lies:
// read before (2^16 packets of 1200 bytes 28 against 31 us, of 2000 bytes 43
// against 48 us), written by a copy just before (25.7 against 23.8 and 48.0 against
// 41.0 us), written by the encoder just before or in HBM (equal within 3%).  2^19
// packets, which the cache cannot hold, take 2-3% longer with ordinary loads (1200
// bytes 224 against 219 us, 2000 bytes 345 against 339 us).
constexpr uint64_t kSegCachedBytes = uint64_t(128) << 20;

// Launches the decode or encode of n_packets with the configured (or
// automatic) group size.
template <bool DECODE>
void launch(const SegArgs& a0, uint32_t n_packets, uint32_t max_msg_bytes, hipStream_t stream)
{
    SegArgs a = a0;
    a.cached = uint64_t(n_packets) * max_msg_bytes <= kSegCachedBytes ? 1u : 0u;
    uint32_t group = g_seg_threads.load();
    if (group == 0) group = auto_threads_per_packet(n_packets, max_msg_bytes);
    const uint32_t per_block = 64 * kSegWaves / group;
    void (*kernel)(SegArgs);
    size_t lds;
    if (group == 256 || (group < 64 && max_msg_bytes < kPartMinBytes)) {
        kernel = group == 8    ? window_kernel<8, DECODE>()
                 : group == 16 ? window_kernel<16, DECODE>()
                 : group == 32 ? window_kernel<32, DECODE>()
                               : window_kernel<256, DECODE>();
        lds = size_t(per_block) * (a.slice_words + kAccWords) * 8;
    } else {
        kernel = group == 8    ? part_kernel<8, DECODE>(max_msg_bytes)
                 : group == 16 ? part_kernel<16, DECODE>(max_msg_bytes)
                 : group == 32 ? part_kernel<32, DECODE>(max_msg_bytes)
                               : part_kernel<64, DECODE>(max_msg_bytes);
        a.slot_dwords = part_slot_dwords(max_msg_bytes, group, a.slice_words);
        a.run_words = (block_capacity(64u / group * a.slot_dwords - kPartSlack - 64u) - kPartEnds) / 2u;
        lds = size_t(per_block) * a.slot_dwords * 4;
    }
    // one launch per slice of packets that fits a dispatch's 32-bit work-item
    // count; a slice addresses its packets through offset descriptor and
    // status pointers (syndromes are placed by each descriptor's seg_off)
    const uint64_t per_launch = hm::max_launch_blocks(64 * kSegWaves) * per_block;
    for (uint64_t first = 0; first < n_packets; first += per_launch) {
        SegArgs s = a;
        s.descs = a.descs + first;
        s.status = a.status ? a.status + first : nullptr;
        s.n_packets = uint32_t(n_packets - first < per_launch ? n_packets - first : per_launch);
        const uint32_t blocks = (s.n_packets + per_block - 1) / per_block;
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * kSegWaves), lds, stream, s);
    }
}

int check_common(const void* enc, const void* descs, uint32_t n_packets, const void* msg, uint32_t max_msg_bytes)
{
    if (n_packets > HAMMING_MAX_BATCH) return HAMMING_ERANGE;
    if (max_msg_bytes < 1 || max_msg_bytes > HAMMING_SEG_MAX_BYTES) return HAMMING_EINVAL;
    if (n_packets == 0) return HAMMING_OK;
    if (!enc || !descs || !msg) return HAMMING_EINVAL;
    if ((reinterpret_cast<uintptr_t>(enc) & 7u) || (reinterpret_cast<uintptr_t>(msg) & 7u) ||
        (reinterpret_cast<uintptr_t>(descs) & 7u))
        return HAMMING_EALIGN;
    return HAMMING_OK;
}

}  // namespace

extern "C" {

int64_t hamming_seg_layout(uint32_t msg_bytes, uint32_t t, uint32_t* k_out, uint32_t* r_out)
{
    if (t < 1 || t > HAMMING_SEG_MAX_T || msg_bytes < 1 || msg_bytes > HAMMING_SEG_MAX_BYTES || 8ull * msg_bytes < t)
        return -1;
    const uint32_t bits = 8u * msg_bytes;
    if ((bits + t - 1) / t > HAMMING_SEG_MAX_K) return -1;
    int64_t total = 0;
    for (uint32_t i = 0; i < t; ++i) {
        const uint32_t k = bits / t + (i < bits % t ? 1u : 0u);
        const uint32_t r = seg_checksum_bits(k);
        if (k_out) k_out[i] = k;
        if (r_out) r_out[i] = r;
        total += int64_t(k) + r;
    }
    return total;
}

int hamming_seg_config_set(uint32_t threads_per_packet)
{
    if (threads_per_packet != 0 && threads_per_packet != 8 && threads_per_packet != 16 && threads_per_packet != 32 &&
        threads_per_packet != 64 && threads_per_packet != 256)
        return HAMMING_EINVAL;
    g_seg_threads.store(threads_per_packet);
    return HAMMING_OK;
}

int hamming_seg_config_get(uint32_t* threads_per_packet)
{
    if (!threads_per_packet) return HAMMING_EINVAL;
    *threads_per_packet = g_seg_threads.load();
    return HAMMING_OK;
}

int hamming_decode_segmented(const uint64_t* enc_arena, uint64_t enc_words, const hamming_seg_packet* descs,
                             uint32_t n_packets, uint32_t max_msg_bytes, uint64_t* msg_arena, uint64_t msg_words,
                             uint16_t* syndromes, uint64_t syndrome_count, uint8_t* status, hipStream_t stream)
{
    int rc = check_common(enc_arena, descs, n_packets, msg_arena, max_msg_bytes);
    if (rc != HAMMING_OK || n_packets == 0) return rc;
    if (syndromes && (reinterpret_cast<uintptr_t>(syndromes) & 1u)) return HAMMING_EALIGN;
    SegArgs a{enc_arena, enc_words, descs, n_packets, max_msg_bytes, msg_arena, msg_words,
              syndromes, syndromes ? syndrome_count : 0, status, msg_slice_words(max_msg_bytes), 0, 0, 0};
    launch<true>(a, n_packets, max_msg_bytes, stream);
    return hipGetLastError() == hipSuccess ? HAMMING_OK : HAMMING_EDEVICE;
}

int hamming_encode_segmented(const uint64_t* msg_arena, uint64_t msg_words, const hamming_seg_packet* descs,
                             uint32_t n_packets, uint32_t max_msg_bytes, uint64_t* enc_arena, uint64_t enc_words,
                             hipStream_t stream)
{
    int rc = check_common(enc_arena, descs, n_packets, msg_arena, max_msg_bytes);
    if (rc != HAMMING_OK || n_packets == 0) return rc;
    SegArgs a{enc_arena, enc_words, descs, n_packets, max_msg_bytes, const_cast<uint64_t*>(msg_arena), msg_words,
              nullptr, 0, nullptr, enc_slice_words(max_msg_bytes), 0, 0, 0};
    launch<false>(a, n_packets, max_msg_bytes, stream);
    return hipGetLastError() == hipSuccess ? HAMMING_OK : HAMMING_EDEVICE;
}

}  // extern "C"
