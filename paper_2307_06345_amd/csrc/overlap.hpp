// Index arithmetic of the comparison of two cornerstone arrays, in plain C++
// (constexpr functions run on the device and on the host).
#pragma once

#include <cstdint>

namespace cs {

// The keys of the old array that a tile of the new one needs: `first` .. `last`,
// from the old leaf around the tile's first key on. p0, p1: the lower bounds of
// the tile's first key and of the key after it, at most the old array's number
// of leaves (at least 1). The new array may be no tree (one of keys that are not
// sorted yet), so p0 and p1 may come in any order: there is always a whole leaf,
// and always inside the old array.
struct OldKeys {
    uint32_t first, last;
};
constexpr OldKeys old_keys(uint32_t p0, uint32_t p1) {
    const uint32_t first = p0 ? p0 - 1 : 0;
    return {first, p1 > first ? p1 : first + 1};
}

// Last index in [lo, hi) of a sorted array whose key is <= k (lo if none; lo <= hi).
template <class A>
constexpr uint32_t at_or_before(const A& a, uint32_t lo, uint32_t hi, uint64_t k) {
    const uint32_t first = lo;
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] <= k)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo > first ? lo - 1 : first;
}

}  // namespace cs
