// Host check of the LDS accesses of the chunk-2^14 rotation with stages between lanes: the one map it
// uses in both directions puts every coordinate where it is looked for, no thread touches a word that
// another thread may not have read yet without a barrier, and every pattern is free of bank
// conflicts under the rules of layout_check.cpp.
#include <cstdio>
#include <set>

#include "thc_layout14.h"

using namespace thc::lay14;

static int bad = 0;
#define CHECK(c, ...) do { if (!(c)) { if (bad < 20) { printf(__VA_ARGS__); printf("\n"); } ++bad; } } while (0)

template <typename F>
static void columns(const char* what, F unit, bool load) {   // 128-bit accesses; F(lane) -> 16-byte unit
    for (int g = 0; g < 64; g += load ? 32 : 8)
        for (int parity = 0; parity < (load ? 2 : 1); ++parity) {
            std::set<uint32_t> s;
            int lanes = 0;
            for (int l = g; l < g + (load ? 32 : 8); ++l) {
                if (load && (((l >> 2) ^ (l >> 3) ^ (l >> 4)) & 1) != parity) continue;
                s.insert(unit(l) & (load ? 15u : 7u));
                ++lanes;
            }
            CHECK((int)s.size() == lanes, "%s: %d lanes from %d on %d columns", what, lanes, g, (int)s.size());
        }
}
template <typename F>
static void banks(const char* what, F word) {
    for (int g = 0; g < 64; g += 32) {
        std::set<uint32_t> s;
        for (int l = g; l < g + 32; ++l) s.insert(word(l) & 31u);
        CHECK(s.size() == 32, "%s: bank conflict in lanes %d..", what, g);
    }
}

int main() {
    // each exchange partner differs in exactly one of i5..i8
    const uint32_t step[4] = {1, 2, 7, 15};
    std::set<uint32_t> blocks;
    for (uint32_t l = 0; l < 64; ++l) {
        blocks.insert(block_of_lane(l));
        for (int k = 0; k < 4; ++k)
            CHECK((block_of_lane(l) ^ block_of_lane(l ^ step[k])) == 1u << k, "lane %u, exchange %d", l, k);
    }
    CHECK(blocks.size() == 64, "blocks of a wave");
    // L1 (permuted) -> L3: coordinate by coordinate, once over the whole buffer, inside the wave's own part
    std::set<uint32_t> seen;
    for (uint32_t wave = 0; wave < 8; ++wave)
        for (uint32_t l = 0; l < 64; ++l)
            for (uint32_t r = 0; r < 32; ++r) {
                const uint32_t i = (wave << 11) | (block_of_lane(l) << 5) | r;
                const uint32_t at = 4 * x3e_load_unit(wave, block_of_lane(l), r >> 2) + (r & 3);
                CHECK(at >> 11 == wave, "stored outside the wave's part");
                seen.insert(at);
                const uint32_t lane3 = ((i >> 5) & 3) | ((i & 15) << 2), wave3 = ((i >> 4) & 1) | (((i >> 7) & 3) << 1);
                CHECK(x3e_store(wave3, lane3, i >> 9) == at, "coordinate %u is read elsewhere", i);
            }
    CHECK(seen.size() == 16384, "not a bijection");
    for (uint32_t wave = 0; wave < 8; ++wave) {
        for (uint32_t q = 0; q < 8; ++q) {
            columns("L1 store", [&](int l) { return x3e_load_unit(wave, block_of_lane(l), q); }, false);
            columns("L4e load", [&](int l) { return x3e_load_unit(wave, block_of_lane(l), q); }, true);
        }
        for (uint32_t r = 0; r < 32; ++r) banks("L3 load and store", [&](int l) { return x3e_store(wave, l, r); });
    }
    // fp32 staging
    std::set<uint32_t> units;
    for (uint32_t u = 0; u < 512; ++u) units.insert(stage_unit(u));
    CHECK(units.size() == 512 && *units.rbegin() == 511, "staging is no bijection");
    for (uint32_t j = 0; j < 8; ++j) {
        columns("stage store", [&](int l) { return stage_unit(j * 64 + l); }, false);
        columns("stage load", [&](int l) { return stage_unit(8 * block_of_lane(l) + j); }, true);
    }
    printf("layout check: %d problems\n", bad);
    return bad != 0;
}
