// Bit-plane input layout: the index-set clustering of Sec. III.A (Fig. 4)
// taken to single positions.  Plane p-1 holds position p of every codeword
// (codeword i at bit i%64 of 64-bit word i/64), so a codeword occupies n bits
// of input instead of one or two padded 64-bit words, and a lane that loads
// one 32-bit word of each plane holds 32 codewords bit-sliced:
//   checksum bit j of all 32 codewords = XOR of the planes in index set I_j
//   (Algorithm 1 applied to 32 codewords at once);
//   correction mask of position p = AND over j of (s_j or ~s_j as bit j of p
//   says), built from two half-width minterm tables;
//   message bit m of the 32 codewords = corrected plane of its position.
// A 32x32 bit transpose turns message planes into per-codeword messages,
// which are packed into the same dense stream as the plain decode and
// written through LDS with coalesced stores; errpos bytes come from the
// syndrome planes with a multiply-spread.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hamming.h"
#include "hamming_device.h"
#include "tile.h"

namespace hm {
namespace {

constexpr bool is_pow2(int p) { return (p & (p - 1)) == 0; }

// Message positions in order (1-based positions, powers of two skipped).
template <int R>
struct MsgPositions {
    int v[Code<R>::K];
    constexpr MsgPositions() : v()
    {
        int c = 0;
        for (int p = 1; p <= Code<R>::N; ++p)
            if (!is_pow2(p)) v[c++] = p;
    }
};

template <int R>
struct PlaneShape {
    static constexpr int N = Code<R>::N;
    static constexpr int K = Code<R>::K;
    static constexpr int NB = (K + 31) / 32;                     // 32-row transpose blocks
    static constexpr int WAVES = 4;                              // waves per block
    // Lanes whose messages are staged at once.  A lane produces K dwords; a
    // buffer for all 64 lanes costs 14.3 KB per wave at r = 6 and 30 KB at
    // r = 7 and left 9 and 5 waves on a CU, so the long messages go out in two
    // rounds of 32 lanes (r = 6, 2^26 codewords: 195 -> 184 us; r = 7, 3.3e7: 279 ->
    // 225 us).  At r = 7 the registers allow 8 waves on a CU, and so do 15 KB for
    // each: four rounds of 16 lanes were no faster at any size (225 us) and made the
    // smallest packets slower (2 MiB of planes 12.1 us against 10.6 with two rounds
    // and 11.4 with one for all lanes).
    static constexpr int LANES = R >= 6 ? 32 : 64;
    static constexpr int MSG_DW = LANES * K;
    static constexpr int EP_DW = 64 * 8;                          // errpos dwords per wave, staged first
    static constexpr int LDS_DW = MSG_DW > EP_DW ? MSG_DW : EP_DW;
    static_assert(MSG_DW % 4 == 0 && LDS_DW % 4 == 0, "staged messages must be whole 16-byte vectors");
};

// In-place transpose of a 32x32 bit matrix: bit c of row i moves to bit i of
// row c.  Stage j exchanges, for rows k and k+j (bit j of k clear), the
// columns with bit j set in row k against the columns with bit j clear in row
// k+j.  Stages 16 and 8 move whole bytes (one byte permute per row), the
// others take a shift and a bit-field insert per row: 256 VALU instructions
// against 480 for the usual masked-difference form of every stage.
__device__ __forceinline__ void transpose32(uint32_t* A)
{
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t x = A[k], y = A[k + 16];
        A[k] = __builtin_amdgcn_perm(y, x, 0x05040100u);        // low halves of x, y
        A[k + 16] = __builtin_amdgcn_perm(y, x, 0x07060302u);   // high halves
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        if (k & 8) continue;
        const uint32_t x = A[k], y = A[k + 8];
        A[k] = __builtin_amdgcn_perm(y, x, 0x06020400u);        // even bytes of x, y interleaved
        A[k + 8] = __builtin_amdgcn_perm(y, x, 0x07030501u);    // odd bytes
    }
    constexpr uint32_t masks[3] = {0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int st = 0; st < 3; ++st) {
        const int j = 4 >> st;
        const uint32_t m = masks[st];
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            if (k & j) continue;
            const uint32_t x = A[k], y = A[k + j];
            A[k] = (x & m) | ((y << j) & ~m);
            A[k + j] = ((x >> j) & m) | (y & ~m);
        }
    }
}

// Blocks of the decode that each XCD takes in turn: neighbouring waves read
// neighbouring 256-byte pieces of every plane, and planes that do not start on
// a cache line share lines between them (2^24 codewords, slices of 16 against
// 1: r = 5 26-28 against 30-32 us, r = 6 48-53 against 57-61 us).
constexpr uint32_t kPlanesXcdChunk = 16;

// Planes of at most this many bytes are read with ordinary loads, larger ones
// with nontemporal loads.  Off whole 128-byte lines two waves share the lines at the
// ends of their pieces, and the caches answer the second (32 MiB of planes just
// written, ordinary against nontemporal loads: r = 4 13.9 against 17.7 us, r = 5 12.9
// against 17.4; from HBM 16.9 against 17.6 and 16.1 either way).  On whole lines
// planes decoded again come out of the Infinity Cache (r = 5 9.8 against 14.7, r = 6
// 11.6 against 15.4), from HBM r = 3 takes 14.5 against 18.2 and the others the same
// within 3%, but just written they take longer (r = 3 14.3 against 11.2, r = 4 13.7
// against 13.0, r = 5 12.2 against 11.4, r = 6 13.7 against 13.0).  Beyond, nontemporal
// ones are 3-10% faster either way (r = 6, 2^24 codewords: 48 against 52-55 us).
constexpr uint64_t kPlanesCachedBytes = uint64_t(64) << 20;

template <int R, bool NT>
__global__ __launch_bounds__(64 * PlaneShape<R>::WAVES) void decode_planes_kernel(
    const uint32_t* __restrict__ planes, uint64_t plane_dwords, uint64_t n_cw, uint32_t* __restrict__ data,
    uint64_t data_dwords, uint8_t* __restrict__ errpos, uint32_t flags)
{
    using S = PlaneShape<R>;
    constexpr int N = S::N, K = S::K, NB = S::NB;
    __shared__ u32x4 lds_raw[S::WAVES * S::LDS_DW / 4];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t wave = uint64_t(xcd_block(blockIdx.x, gridDim.x, kPlanesXcdChunk)) * S::WAVES + wib;
    const uint64_t groups = (n_cw + 31) / 32;
    if (wave * 64 >= groups) return;
    const uint64_t g = wave * 64 + lane;
    uint32_t* buf = reinterpret_cast<uint32_t*>(lds_raw) + wib * S::LDS_DW;

    // a1: one dword of every plane = 32 codewords, bit-sliced
    uint32_t P[N];
    if (g < groups) {
        const uint32_t* src = planes + g;
#pragma unroll
        for (int p = 0; p < N; ++p) {
            if constexpr (NT)
                P[p] = __builtin_nontemporal_load(src + uint64_t(p) * plane_dwords);
            else
                P[p] = src[uint64_t(p) * plane_dwords];
        }
        if (g == groups - 1 && (n_cw & 31u)) {
            const uint32_t valid = (1u << (n_cw & 31u)) - 1u;
#pragma unroll
            for (int p = 0; p < N; ++p) P[p] &= valid;
        }
    } else {
#pragma unroll
        for (int p = 0; p < N; ++p) P[p] = 0;
    }

    // a2: checksum planes
    uint32_t s[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        uint32_t x = 0;
#pragma unroll
        for (int p = 1; p <= N; ++p)
            if ((p >> j) & 1) x ^= P[p - 1];
        s[j] = x;
    }

    // a3: errpos bytes, codeword c = byte c%4 of dword c/4, out through the
    // wave's buffer before the messages need it
    if (errpos) {
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            uint32_t e = 0;
#pragma unroll
            for (int j = 0; j < R; ++j) e |= ((((s[j] >> (4 * d)) & 0xFu) * 0x00204081u) & 0x01010101u) << j;
            buf[lane * 8 + d] = e;
        }
        wave_sync();
        const uint64_t e0 = wave * 2048;
        const bool ev = (flags & kFlagEpVec) != 0;
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            const uint32_t v = lane + 64 * q;
            const uint64_t at = e0 + 16ull * v;
            if (at >= n_cw) break;
            const u32x4 x = *reinterpret_cast<const u32x4*>(buf + 4 * v);
            if (ev && at + 16 <= n_cw) {
                __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(errpos + at));
            } else {
                for (int i = 0; i < 16 && at + i < n_cw; ++i) errpos[at + i] = uint8_t(x[i / 4] >> (8 * (i % 4)));
            }
        }
        wave_sync();
    }

    // a4: correction masks from minterms of the low and high checksum planes
    constexpr int H = R / 2, HH = R - H;
    uint32_t lo[1 << H], hi[1 << HH];
    lo[0] = ~s[0];
    lo[1] = s[0];
#pragma unroll
    for (int j = 1; j < H; ++j) {
#pragma unroll
        for (int a = (1 << j) - 1; a >= 0; --a) {
            lo[a | (1 << j)] = lo[a] & s[j];
            lo[a] &= ~s[j];
        }
    }
    hi[0] = ~s[H];
    hi[1] = s[H];
#pragma unroll
    for (int j = 1; j < HH; ++j) {
#pragma unroll
        for (int a = (1 << j) - 1; a >= 0; --a) {
            hi[a | (1 << j)] = hi[a] & s[H + j];
            hi[a] &= ~s[H + j];
        }
    }

    // a5: corrected message planes, padded to whole transpose blocks
    constexpr MsgPositions<R> kPos{};
    uint32_t X[NB * 32];
#pragma unroll
    for (int m = 0; m < NB * 32; ++m) {
        if (m < K) {
            constexpr int kLoMask = (1 << H) - 1;
            const int p = kPos.v[m];
            X[m] = P[p - 1] ^ (lo[p & kLoMask] & hi[p >> H]);
        } else {
            X[m] = 0;
        }
    }
    uint32_t out[K];                 // the lane's 32 messages in stream order
    if constexpr (K == 4) {
        // Hamming(7,4): output dword w holds codewords 8w..8w+7, four bits
        // each; spread byte w of message plane m to every fourth bit
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            out[w] = 0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                uint32_t x = (X[m] >> (8 * w)) & 0xFFu;
                x = (x | (x << 12)) & 0x000F000Fu;
                x = (x | (x << 6)) & 0x03030303u;
                x = (x | (x << 3)) & 0x11111111u;
                out[w] |= x << m;
            }
        }
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b) transpose32(X + 32 * b);

        // a6: codeword c's message bits [32b, 32b+32) are X[32b + c]; append
        // them in stream order (c*K + 32b), completing one dword after another
        uint32_t acc = 0;
        int filled = 0, wout = 0;
#pragma unroll
        for (int c = 0; c < 32; ++c) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t v = X[32 * b + c];
                const int len = (K - 32 * b) < 32 ? (K - 32 * b) : 32;
                acc |= filled ? (v << filled) : v;
                if (filled + len >= 32) {
                    out[wout] = acc;
                    ++wout;
                    acc = filled ? (v >> (32 - filled)) : 0u;
                    filled = filled + len - 32;
                } else {
                    filled += len;
                }
            }
        }
    }

    // LANES lanes at a time: their messages are one contiguous piece of the
    // stream, staged in LDS and stored in 16-byte vectors by consecutive lanes
#pragma unroll
    for (int round = 0; round < 64 / S::LANES; ++round) {
        if (S::LANES == 64 || lane / S::LANES == uint32_t(round)) {
            const uint32_t l = lane % S::LANES;
            if constexpr (K % 4 == 0) {
#pragma unroll
                for (int w = 0; w < K; w += 4)
                    *reinterpret_cast<u32x4*>(buf + l * K + w) = u32x4{out[w], out[w + 1], out[w + 2], out[w + 3]};
            } else {
#pragma unroll
                for (int w = 0; w < K; ++w) buf[l * K + w] = out[w];
            }
        }
        wave_sync();
        const uint64_t dw0 = (wave * 64 + round * S::LANES) * K;
#pragma unroll
        for (uint32_t q = 0; q < (S::MSG_DW / 4 + 63) / 64; ++q) {
            const uint32_t v = lane + 64 * q;
            if (v >= uint32_t(S::MSG_DW / 4)) break;
            const uint64_t at = dw0 + 4ull * v;
            const u32x4 x = *reinterpret_cast<const u32x4*>(buf + 4 * v);
            if (at + 4 <= data_dwords) {
                __builtin_nontemporal_store(x, reinterpret_cast<u32x4a8*>(data + at));
            } else {
                for (int i = 0; i < 4 && at + i < data_dwords; ++i) data[at + i] = x[i];
            }
        }
        wave_sync();
    }
}

// Natural layout -> planes.  A wave converts 2048 consecutive codewords, 32
// per lane, one storage dword at a time: the words arrive as 16-byte vectors
// by consecutive lanes (coalesced), pass through LDS to the lane that owns
// them, and a lane's 32 dwords are transposed in registers into one dword of
// each of 32 planes, so every store writes 256 contiguous bytes of a plane.
// Only the dwords that hold positions are staged (one of two for r <= 5), in
// an 8 KB buffer per wave that the dwords of a codeword take in turn.
// 16-byte slots are rotated per block of eight, so a lane's reads (128 bytes
// apart from its neighbours') spread over the banks.
//
// Bound by HBM.  The first form (a lane loading its 32 codewords itself, 4
// bytes at a 256-byte lane stride) spent its time on the 64 cache lines that
// each load touched: 82 us (r = 5) and 130 us (r = 6) for 2^24 codewords,
// against 35 and 46 us now (5.7 TB/s).  Consecutive blocks go to one
// XCD in slices of 32 (1: 3-8% slower at 2^24 codewords, equal at 2^26).
//
// NT: nontemporal plane stores.  They are 4-7% faster when every plane starts
// on a 128-byte line, so that a wave's 256 bytes are whole lines (r = 6, 2^24
// codewords: 46.8 against 49.7 us); otherwise two waves share the lines at
// the ends of their pieces, and plain stores, which the L2 merges, win by 4-16%
// (r = 7: 115 against 137 us).
constexpr int kToPlanesWaves = 4;
constexpr uint32_t kToPlanesXcdChunk = 32;
constexpr uint32_t kToPlanesCw = 2048;        // codewords per wave

template <int R, bool NT>
__global__ __launch_bounds__(64 * kToPlanesWaves) void to_planes_kernel(const uint64_t* __restrict__ cw,
                                                                        uint64_t n_cw,
                                                                        uint32_t* __restrict__ planes,
                                                                        uint64_t plane_dwords)
{
    constexpr int N = Code<R>::N, WPC = Code<R>::WPC;
    constexpr int ND = (N + 31) / 32;         // storage dwords that hold positions
    constexpr int NV = 16 * WPC;              // 16-byte vectors per lane
    constexpr int PER = 2 / WPC;              // codewords per vector
    __shared__ u32x4 lds_raw[kToPlanesWaves][kToPlanesCw / 4];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t wave = uint64_t(xcd_block(blockIdx.x, gridDim.x, kToPlanesXcdChunk)) * kToPlanesWaves + wib;
    if (wave * kToPlanesCw >= n_cw) return;
    uint32_t* buf = reinterpret_cast<uint32_t*>(&lds_raw[wib][0]);

    // All loads are in flight before the first is used.  A check of its own per
    // vector made each wait for the one before (2^18 codewords of r = 5 from HBM 10.2 us
    // against 4.3; 2^22 13.3 against 11.2).
    uint32_t in[NV][PER][ND];
    const uint64_t* words = cw + wave * kToPlanesCw * WPC;
    const uint64_t rem = (n_cw - wave * kToPlanesCw) * WPC;      // input words left
    u32x4 x[NV];
    if (rem >= uint64_t(kToPlanesCw) * WPC) {
        const u32x4a8* src = reinterpret_cast<const u32x4a8*>(words) + lane;
#pragma unroll
        for (int v = 0; v < NV; ++v) x[v] = __builtin_nontemporal_load(src + 64 * v);
    } else {
        // words past the last one are read as the last one, and zeroed
        const uint32_t last = uint32_t(rem) - 1u;
        uint64_t y[NV][2];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t w = 2u * (64u * v + lane);            // first word of this lane's vector v
            y[v][0] = words[min(w, last)];
            y[v][1] = words[min(w + 1u, last)];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t w = 2u * (64u * v + lane);
            const uint64_t lo = w <= last ? y[v][0] : 0, hi = w + 1u <= last ? y[v][1] : 0;
            x[v] = u32x4{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
        }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int c = 0; c < PER; ++c)
#pragma unroll
            for (int d = 0; d < ND; ++d) in[v][c][d] = x[v][c * 2 * WPC + d];

    const uint64_t g = wave * 64 + lane;
    const bool stores = 32 * g < n_cw;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        if (d > 0) wave_sync();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t c = (64u * v + lane) * PER;           // first codeword of the vector
            const uint32_t slot = c / 4;
            uint32_t* at = buf + 4 * (slot ^ ((slot >> 3) & 7u)) + c % 4;
            if constexpr (PER == 2)
                *reinterpret_cast<uint2*>(at) = make_uint2(in[v][0][d], in[v][1][d]);
            else
                *at = in[v][0][d];
        }
        wave_sync();
        uint32_t A[32];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            const u32x4 x = *reinterpret_cast<const u32x4*>(buf + 4 * (8 * lane + (q ^ (lane & 7u))));
            A[4 * q + 0] = x.x;
            A[4 * q + 1] = x.y;
            A[4 * q + 2] = x.z;
            A[4 * q + 3] = x.w;
        }
        transpose32(A);
        if (stores) {
            uint32_t* dst = planes + uint64_t(32 * d) * plane_dwords + g;
#pragma unroll
            for (int b = 0; b < 32; ++b) {
                if (32 * d + b >= N) break;
                if constexpr (NT)
                    __builtin_nontemporal_store(A[b], dst + uint64_t(b) * plane_dwords);
                else
                    dst[uint64_t(b) * plane_dwords] = A[b];
            }
        }
    }
}

template <int R>
void launch_planes(const uint64_t* planes, uint64_t plane_words, uint64_t n_cw, void* data, uint8_t* errpos,
                   uint32_t flags, hipStream_t stream)
{
    using S = PlaneShape<R>;
    const uint64_t waves = ((n_cw + 31) / 32 + 63) / 64;
    const uint64_t blocks = (waves + S::WAVES - 1) / S::WAVES;
    const uint64_t data_dwords = hamming_data_bytes(n_cw, R) / 4;
    void (*const kernel)(const uint32_t*, uint64_t, uint64_t, uint32_t*, uint64_t, uint8_t*, uint32_t) =
        uint64_t(Code<R>::N) * n_cw / 8 > kPlanesCachedBytes ? decode_planes_kernel<R, true>
                                                             : decode_planes_kernel<R, false>;
    hipLaunchKernelGGL(kernel, dim3(uint32_t(blocks)), dim3(64 * S::WAVES), 0, stream,
                       reinterpret_cast<const uint32_t*>(planes), plane_words * 2, n_cw,
                       static_cast<uint32_t*>(data), data_dwords, errpos, flags);
}

template <int R>
void launch_to_planes(const uint64_t* cw, uint64_t n_cw, uint64_t* planes, uint64_t plane_words, hipStream_t stream)
{
    const uint64_t groups = (n_cw + 31) / 32;
    const bool whole_lines = ((reinterpret_cast<uintptr_t>(planes) | (plane_words * 8)) & 127u) == 0;
    void (*const kernel)(const uint64_t*, uint64_t, uint32_t*, uint64_t) =
        whole_lines ? to_planes_kernel<R, true> : to_planes_kernel<R, false>;
    hipLaunchKernelGGL(kernel, dim3(uint32_t((groups + 255) / 256)), dim3(64 * kToPlanesWaves), 0, stream, cw, n_cw,
                       reinterpret_cast<uint32_t*>(planes), plane_words * 2);
}

}  // namespace
}  // namespace hm

extern "C" {

// One launch covers at most this many codewords: both plane kernels then
// stay within a dispatch's 32-bit work-item count (one lane per 32 codewords).
constexpr uint64_t kPlanesMaxCodewords = (uint64_t(1) << 37) - (uint64_t(1) << 13);

uint64_t hamming_planes_words(uint64_t n_cw, int r)
{
    if (r < 3 || r > 7 || n_cw > HAMMING_MAX_CODEWORDS) return 0;
    return uint64_t((1 << r) - 1) * ((n_cw + 63) / 64);
}

int hamming_decode_planes(const uint64_t* planes, uint64_t plane_words, uint64_t n_cw, int r, void* data_out,
                          uint8_t* errpos_out, hipStream_t stream)
{
    if (r < 3 || r > 7) return HAMMING_EINVAL;
    if (n_cw > kPlanesMaxCodewords) return HAMMING_ERANGE;
    if (n_cw == 0) return HAMMING_OK;
    if (!planes || !data_out) return HAMMING_EINVAL;
    if (plane_words < (n_cw + 63) / 64) return HAMMING_ERANGE;
    if ((reinterpret_cast<uintptr_t>(planes) & 7u) || (reinterpret_cast<uintptr_t>(data_out) & 7u))
        return HAMMING_EALIGN;
    uint32_t flags = 0;
    if (errpos_out && !(reinterpret_cast<uintptr_t>(errpos_out) & 15u)) flags |= hm::kFlagEpVec;
    switch (r) {
    case 3: hm::launch_planes<3>(planes, plane_words, n_cw, data_out, errpos_out, flags, stream); break;
    case 4: hm::launch_planes<4>(planes, plane_words, n_cw, data_out, errpos_out, flags, stream); break;
    case 5: hm::launch_planes<5>(planes, plane_words, n_cw, data_out, errpos_out, flags, stream); break;
    case 6: hm::launch_planes<6>(planes, plane_words, n_cw, data_out, errpos_out, flags, stream); break;
    default: hm::launch_planes<7>(planes, plane_words, n_cw, data_out, errpos_out, flags, stream); break;
    }
    return hipGetLastError() == hipSuccess ? HAMMING_OK : HAMMING_EDEVICE;
}

int hamming_to_planes(const uint64_t* codewords, uint64_t n_cw, int r, uint64_t* planes, uint64_t plane_words,
                      hipStream_t stream)
{
    if (r < 3 || r > 7) return HAMMING_EINVAL;
    if (n_cw > kPlanesMaxCodewords) return HAMMING_ERANGE;
    if (n_cw == 0) return HAMMING_OK;
    if (!codewords || !planes) return HAMMING_EINVAL;
    if (plane_words < (n_cw + 63) / 64) return HAMMING_ERANGE;
    if ((reinterpret_cast<uintptr_t>(codewords) & 7u) || (reinterpret_cast<uintptr_t>(planes) & 7u))
        return HAMMING_EALIGN;
    switch (r) {
    case 3: hm::launch_to_planes<3>(codewords, n_cw, planes, plane_words, stream); break;
    case 4: hm::launch_to_planes<4>(codewords, n_cw, planes, plane_words, stream); break;
    case 5: hm::launch_to_planes<5>(codewords, n_cw, planes, plane_words, stream); break;
    case 6: hm::launch_to_planes<6>(codewords, n_cw, planes, plane_words, stream); break;
    default: hm::launch_to_planes<7>(codewords, n_cw, planes, plane_words, stream); break;
    }
    return hipGetLastError() == hipSuccess ? HAMMING_OK : HAMMING_EDEVICE;
}

}  // extern "C"
