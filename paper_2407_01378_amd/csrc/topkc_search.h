// The search of a workgroup in the ascending list of selected chunks: `probes` positions at a time cut what is
// left of it to 1/probes (a halving search is a chain of 18 dependent reads for a quarter million of entries).
// The list may have any number of entries a 32-bit count can tell, so sums of positions are 64 bits wide.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define THC_SEARCH_HD __host__ __device__ __forceinline__
#else
#define THC_SEARCH_HD inline
#endif

namespace thc {

// A chunk's place in the list, or that it has none: a list of up to 2^32 - 1 entries has no such place.
constexpr uint32_t kNotSelected = 0xFFFFFFFFu;
THC_SEARCH_HD bool is_selected(uint32_t place) { return place != kNotSelected; }

// Entries in front of lo are below the bound that is looked for, entry hi (or the end of the list) is not.
struct SearchRange {
    uint32_t lo, hi;
    THC_SEARCH_HD uint32_t step(uint32_t probes) const { return (hi - lo - 1u) / probes + 1u; }   // lo < hi
    // Position that probe t looks at; from hi on there is nothing to look at.
    THC_SEARCH_HD uint64_t at(uint32_t t, uint32_t step) const { return (uint64_t)lo + (uint64_t)t * step; }
    // What is left once the first `count` probes, and no other, have found entries below the bound.
    THC_SEARCH_HD void cut(uint32_t count, uint32_t step) {
        if (count == 0u) {
            hi = lo;
            return;
        }
        const uint32_t last = (uint32_t)at(count - 1u, step);   // (it has been looked at: below hi)
        if (hi - last > step) hi = last + step;
        lo = last + 1u;
    }
};

}  // namespace thc
