// Every mask of every group of four through both rounds of the sparse matrix product (paper_2502_07590_amd/csrc/pair_slots.h).
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "pair_slots.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "group %d, mask %d, others %x: %s\n", g, mask, others, #c); std::exit(1); } } while (0)

int main()
{
    for (int g = 0; g < 4; ++g)
        for (int mask = 0; mask < 16; ++mask)
            for (unsigned others : {0u, ~0u, 0x5A96C3F0u, 0xA5693C0Fu}) {
                const int at = 2 * (g & 1) + 16 * (g >> 1);  // pair i of the group: bit 4 i + at
                unsigned w = others;
                for (int i = 0; i < 4; ++i) w = (w & ~(1u << (4 * i + at))) | ((unsigned)(mask >> i & 1) << (4 * i + at));
                const dsv::PairSlots ps(w);
                auto bit = [&](uint32_t x) { return (int)(x >> at & 1); };
                const int first = (int)(ps.index >> (4 * g)), left = (int)(ps.index_left() >> (4 * g));
                const int s0 = first & 3, s1 = first >> 2 & 3, t0 = left & 3, t1 = left >> 2 & 3;
                CHECK(s0 < s1);
                CHECK(t0 < t1);
                // the pairs whose scores the kernel picks for the slots
                CHECK(s0 == (bit(ps.b0) ? 0 : bit(ps.b1) ? 1 : 2));
                CHECK(s1 == (bit(ps.n3) ? bit(ps.n2) ? 1 : 2 : 3));
                CHECK(t0 == (bit(ps.r1) ? 1 : 2));
                const bool u0 = bit(ps.r1) | bit(ps.r2), u1 = bit(ps.r1) & bit(ps.r2);
                CHECK(!u1 || t1 == 2);
                // every selected pair once, no other pair at all
                const int sum = (bit(ps.v0) << s0) + (bit(ps.v1) << s1) + ((int)u0 << t0) + ((int)u1 << t1);
                const int any = (bit(ps.v0) << s0) | (bit(ps.v1) << s1) | ((int)u0 << t0) | ((int)u1 << t1);
                CHECK(sum == mask && any == mask);
                CHECK(ps.index >> 16 == 0 && ps.index_left() >> 16 == 0);
            }
    std::puts("pair slots ok");
}
