// Host check of the search in the list of selected chunks (topkc_search.h), lists of up to 2^32 - 1 entries among
// them: entry j is j * stride, so no list is stored.  Compiled and run by tests/test_topkc_search_host.py.
#include <cstdio>
#include <initializer_list>

#include "topkc_search.h"

static int bad = 0;

static void search(uint32_t J, uint64_t stride, uint64_t bound, uint32_t probes) {
    thc::SearchRange r = {0u, J};
    int rounds = 0;
    while (r.lo < r.hi && rounds < 40) {
        const uint32_t step = r.step(probes);
        uint32_t count = 0, outside = 0;
        for (uint32_t t = 0; t < probes; ++t) {
            const uint64_t at = r.at(t, step);
            if (at >= r.hi) { ++outside; continue; }
            if (outside != 0 || at < r.lo) ++bad;      // positions ascend and do not come round again
            if (at * stride < bound) ++count;
        }
        r.cut(count, step);
        ++rounds;
    }
    const uint64_t first = (bound + stride - 1) / stride;
    const uint64_t want = first < J ? first : J;
    if (r.lo != want || r.lo != r.hi || rounds > 7) {
        if (bad < 20) printf("J %u stride %llu bound %llu: found %u, is %llu, %d rounds\n", J, (unsigned long long)stride,
                             (unsigned long long)bound, r.lo, (unsigned long long)want, rounds);
        ++bad;
    }
}

int main() {
    const uint32_t sizes[] = {0u, 1u, 2u, 255u, 256u, 257u, 511u, 65536u, 65537u, 203273u, 0x7FFFFFFFu, 0x80000000u,
                              0xFFFFFE00u, 0xFFFFFEFFu, 0xFFFFFF00u, 0xFFFFFF01u, 0xFFFFFF80u, 0xFFFFFFFEu, 0xFFFFFFFFu};
    for (uint32_t J : sizes)
        for (uint64_t stride : {1ull, 3ull})
            for (uint64_t part = 0; part <= 64; ++part)
                for (uint64_t off : {0ull, 1ull, 2ull, 300ull})
                    for (uint32_t probes : {64u, 256u}) search(J, stride, (J * stride / 64) * part + off, probes);
    for (uint32_t place : {0u, 1u, 0x7FFFFFFFu, 0x80000000u, 0xFFFFFFFEu})   // every place that a list has
        if (!thc::is_selected(place)) ++bad;
    if (thc::is_selected(thc::kNotSelected)) ++bad;
    printf("%d problems\n", bad);
    return bad != 0;
}
