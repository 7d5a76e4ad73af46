// Host checks of the part form's block layout in LDS (seg_parts.h): a run staged
// in blocks reads back at every dword as the flat run does, windows ORed into
// cleared blocks and merged give the flat result, nothing leaves the area, and
// lanes a multiple of 32 dwords apart meet in different banks.  Prints "seg blocks
// ok" and exits 0 when every check holds.
#include <stdint.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "seg_parts.h"

#define CHECK(cond)                                                       \
    do {                                                                  \
        if (!(cond)) {                                                    \
            fprintf(stderr, "line %d: %s (%u)\n", __LINE__, #cond, D);    \
            return 1;                                                     \
        }                                                                 \
    } while (0)

using u32 = uint32_t;
constexpr u32 R = hm::kBlockRoom, B = hm::kBlockDwords;

static int check_area(u32 D, std::mt19937& rng)
{
    const u32 area = hm::block_area(D);
    CHECK(hm::block_capacity(area) <= D && hm::block_capacity(area) + 4 >= D);
    for (u32 l = 0; l < 2 * B; ++l) CHECK(hm::block_area(hm::block_capacity(area + l)) <= area + l);
    std::vector<u32> flat(D + 8, 0), lds(area, 0xDEADBEEF);
    for (u32 a = 0; a < D; ++a) flat[a] = rng();
    for (u32 a = 0; a < D; ++a) {                       // staging, the first of a block twice
        CHECK(hm::block_at(a) < area);
        lds[hm::block_at(a)] = flat[a];
        if (a % B < R && a >= B) lds[hm::block_at(a) - R] = flat[a];
    }
    for (u32 a = 0; a + 5 <= D; ++a)
        for (u32 k = 0; k < 5; ++k) CHECK(lds[hm::block_at(a) + k] == flat[a + k]);

    std::vector<u32> want(D, 0), out(area, 0);
    u32 bit = 0;                                        // runs of bits end to end, as messages and segments lie
    while (bit + 128 + 32 <= 32 * D) {
        u32 x[4] = {u32(rng()), u32(rng()), u32(rng()), u32(rng())};
        const u32 len = 1 + rng() % 128;
        hm::mask_window(x, int32_t(len) - 1);
        for (u32 q = 0; q < len; ++q) want[(bit + q) / 32] |= ((x[q / 32] >> (q % 32)) & 1u) << ((bit + q) % 32);
        const hm::Placed p = hm::place_window(x, bit);
        for (u32 k = 0; k < 5; ++k) {
            const u32 a = u32(p.first) + 8 * B;         // the area's dword 8 B takes bit 0: first may be -1
            const u32 at = hm::block_at(a) + k - hm::block_at(8 * B);
            if (p.first < 0 && k == 0) {
                CHECK(p.y[k] == 0);
                continue;
            }
            const u32 to = p.first < 0 ? k - 1 : at;
            CHECK(to < area || p.y[k] == 0);
            if (to < area) out[to] |= p.y[k];
        }
        bit += len;
    }
    for (u32 b = 1; b * B < D; ++b)
        for (u32 k = 0; k < R; ++k) out[b * (B + R) + k] ^= out[b * (B + R) - R + k];
    for (u32 a = 0; a < D; ++a) CHECK(out[hm::block_at(a)] == want[a]);
    return 0;
}

int main()
{
    std::mt19937 rng(5);
    for (u32 D = 5; D < 700; ++D)
        if (check_area(D, rng)) return 1;
    for (u32 D : {1024u, 2047u, 4096u, 4500u})
        if (check_area(D, rng)) return 1;
    for (u32 step : {32u, 64u, 96u, 160u, 480u}) {      // eight lanes' vectors of four dwords: 32 banks, each once
        const u32 D = step;
        for (u32 a0 = 0; a0 < 32; ++a0) {
            u32 seen = 0;
            for (u32 l = 0; l < 8; ++l) seen |= 1u << (hm::block_at(a0 + l * step) / 4 % 8);
            CHECK(step % 64 == 0 || seen == 0xFF);
        }
    }
    printf("seg blocks ok\n");
    return 0;
}
