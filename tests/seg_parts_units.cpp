// Host checks of the part form's bit work (seg_parts.h): whole packets are
// encoded and decoded lane by lane as the kernels do it, through the same
// functions, and compared with bit-by-bit definitions, for every number of
// lanes per packet.  Prints "seg parts ok" and exits 0 when every check holds.
#include <stdint.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "seg_parts.h"

#define CHECK(cond)                                                                                            \
    do {                                                                                                       \
        if (!(cond)) {                                                                                         \
            fprintf(stderr, "line %d: %s (bytes %u, t %u, lanes %u)\n", __LINE__, #cond, M, t, G);             \
            return 1;                                                                                          \
        }                                                                                                      \
    } while (0)

using u32 = uint32_t;
constexpr u32 kPad = 4, kMaxLen = 12;

static u32 checksum_bits(u32 k)
{
    u32 r = 2;
    while ((1u << r) - 1 - r < k) ++r;
    return r;
}

struct Window {
    u32 i, v, x[4];
};

static int check_packet(u32 M, u32 t, u32 G, std::mt19937& rng)
{
    const u32 bits = 8 * M, q = bits / t, rem = bits % t;
    CHECK(hm::small_div(bits, t) == q);
    const u32 widest = rem ? q + 1 + checksum_bits(q + 1) : q + checksum_bits(q);
    const hm::Parts P = hm::make_parts(t, widest / 128 + 1, G);
    for (u32 l = 0; l < G; ++l) CHECK(P.segment(l) == l / P.parts);
    CHECK(P.parts * t <= G && P.parts * P.len >= widest / 128 + 1);
    if (G == 64) CHECK(P.len <= 6);
    if (P.len > kMaxLen) return 0;

    std::vector<u32> n(t), K(t), o(t);
    u32 total = 0;
    for (u32 i = 0, k0 = 0; i < t; ++i) {
        const u32 k = q + (i < rem ? 1 : 0);
        n[i] = k + checksum_bits(k);
        K[i] = k0;
        o[i] = total;
        k0 += k;
        total += n[i];
    }
    std::vector<char> msg(bits), enc(total);
    for (auto& b : msg) b = char(rng() & 1);
    for (u32 i = 0; i < t; ++i) {
        u32 s = 0, m = 0;
        for (u32 p = 1; p <= n[i]; ++p)
            if (p & (p - 1)) {
                enc[o[i] + p - 1] = msg[K[i] + m++];
                if (enc[o[i] + p - 1]) s ^= p;
            }
        for (u32 p = 1, j = 0; p <= n[i]; p *= 2, ++j) enc[o[i] + p - 1] = char((s >> j) & 1);
    }

    const u32 ew = (total + 63) / 64, mw = (M + 7) / 8;
    std::vector<u32> S(kPad + 2 * ew + 8 + 4 * kMaxLen);
    auto fill = [&](const std::vector<char>& from) {
        for (auto& w : S) w = rng();
        for (u32 b = 0; b < from.size(); ++b) {
            u32& w = S[kPad + b / 32];
            w = (w & ~(1u << (b % 32))) | (u32(from[b]) << (b % 32));
        }
    };
    auto read = [&](u32 dword, u32 sh, u32 (&x)[4]) {
        for (u32 k = 0; k < 4; ++k) x[k] = hm::align32(S.at(dword + k + 1), S.at(dword + k), sh);
    };
    auto put = [&](int32_t base, const hm::Placed& w) {
        for (int k = 0; k < 5; ++k) S.at(size_t(base + w.first + k)) |= w.y[k];
    };

    // encode
    fill(msg);
    std::vector<u32> syn(t, 0);
    std::vector<Window> win;
    for (u32 l = 0; l < G; ++l) {
        const u32 i = P.segment(l), v0 = (l - i * P.parts) * P.len;
        if (i >= t) continue;
        hm::PartSyndrome ps;
        for (u32 v = v0; v < v0 + P.len && v <= n[i] / 128; ++v) {
            Window w{i, v, {}};
            const u32 at = K[i] + (v ? hm::run_base(v) : 0);
            read(kPad + at / 32, at % 32, w.x);
            if (v == 0)
                hm::expand_head(w.x);
            else
                w.x[0] &= ~hm::is_pow2_window(v);
            hm::mask_window(w.x, int32_t(n[i]) - int32_t(128 * v));
            ps.add(w.x, v);
            win.push_back(w);
        }
        syn[i] ^= ps.value();
    }
    for (u32 d = 0; d < 2 * ew + 6; ++d) S[kPad + d] = 0;
    for (const Window& w : win) put(int32_t(kPad) - 1, hm::place_window(w.x, o[w.i] + 128 * w.v + 31));
    for (u32 i = 0; i < t; ++i)
        for (u32 j = 0; (syn[i] >> j) != 0; ++j)
            if ((syn[i] >> j) & 1) {
                const u32 b = o[i] + (1u << j) - 1;
                CHECK(b < o[i] + n[i]);
                S[kPad + b / 32] |= 1u << (b % 32);
            }
    for (u32 b = 0; b < 64 * ew; ++b) CHECK(((S[kPad + b / 32] >> (b % 32)) & 1) == u32(b < total ? enc[b] : 0));

    // decode, with up to two flips per segment
    std::vector<char> got = enc, want;
    for (u32 i = 0; i < t; ++i)
        for (u32 f = rng() % 3; f > 0; --f) got[o[i] + rng() % n[i]] ^= 1;
    fill(got);
    win.clear();
    std::fill(syn.begin(), syn.end(), 0);
    for (u32 l = 0; l < G; ++l) {
        const u32 i = P.segment(l), v0 = (l - i * P.parts) * P.len;
        if (i >= t) continue;
        hm::PartSyndrome ps;
        for (u32 v = v0; v < v0 + P.len && v <= n[i] / 128; ++v) {
            Window w{i, v, {}};
            const u32 b = o[i] + 128 * v + 32 * kPad - 1;
            read(b / 32, b % 32, w.x);
            hm::mask_window(w.x, int32_t(n[i]) - int32_t(128 * v));
            if (v == 0) w.x[0] &= ~1u;
            ps.add(w.x, v);
            win.push_back(w);
        }
        syn[i] ^= ps.value();
    }
    for (u32 i = 0; i < t; ++i) {
        u32 s = 0;
        for (u32 p = 1; p <= n[i]; ++p)
            if (got[o[i] + p - 1]) s ^= p;
        CHECK(syn[i] == s);
        for (u32 p = 1; p <= n[i]; ++p)
            if (p & (p - 1)) want.push_back(got[o[i] + p - 1]);
    }
    for (u32 d = 0; d < 2 * mw + 5; ++d) S[kPad + d] = 0;
    for (Window& w : win) {
        u32 at = K[w.i];
        if (w.v == 0) {
            hm::compact_head(w.x);
        } else {
            w.x[0] &= ~hm::is_pow2_window(w.v);
            at += hm::run_base(w.v);
        }
        put(int32_t(kPad), hm::place_window(w.x, at));
    }
    for (u32 b = 0; b < 64 * mw; ++b) CHECK(((S[kPad + b / 32] >> (b % 32)) & 1) == u32(b < bits ? want[b] : 0));
    return 0;
}

int main()
{
    std::mt19937 rng(7);
    for (u32 G : {8u, 16u, 32u, 64u})
        for (u32 M = 1; M <= 4096; M += M < 80 ? 1 : 61)
            for (u32 t = 1; t <= 32 && t <= 8 * M && t <= G; ++t)
                if (check_packet(M, t, G, rng)) return 1;
    printf("seg parts ok\n");
    return 0;
}
