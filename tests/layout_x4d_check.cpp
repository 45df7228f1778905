// Host check of the decoders' one LDS exchange (X4d, thc_layout14.h): what a wave stores behind its 11
// stages lies where layout L4d looks for it, inside the wave's own 8 KB, once over the whole buffer, and
// both patterns are free of bank conflicts under the rules of layout_check.cpp.
// Compiled and run by tests/test_layout_x4d_host.py.
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

int main() {
    std::set<uint32_t> seen;
    for (uint32_t wave = 0; wave < 8; ++wave)
        for (uint32_t l = 0; l < 64; ++l)
            for (uint32_t q = 0; q < 8; ++q) {
                // the coordinate (i0 = i1 = 0) that the lane holds there behind the two register swaps
                const uint32_t i = ((q & 3u) << 2) | (((l >> 4) & 1u) << 4) | ((block_of_lane(l) & 15u) << 5) |
                                   ((l >> 5) << 9) | ((q >> 2) << 10) | (wave << 11);
                const uint32_t at = x4d_store_unit(wave, l, q);
                CHECK(at >> 9 == wave, "stored outside the wave's part");
                seen.insert(at);
                CHECK(x4d_load_unit((i >> 8) & 7u, (i >> 2) & 63u, i >> 11) == at, "coordinate %u is read elsewhere", i);
            }
    CHECK(seen.size() == 4096 && *seen.rbegin() == 4095, "not a bijection");
    for (uint32_t wave = 0; wave < 8; ++wave)
        for (uint32_t q = 0; q < 8; ++q) {
            columns("store", [&](int l) { return x4d_store_unit(wave, l, q); }, false);
            columns("L4d load", [&](int l) { return x4d_load_unit(wave, l, q); }, true);
        }
    printf("layout check: %d problems\n", bad);
    return bad != 0;
}
