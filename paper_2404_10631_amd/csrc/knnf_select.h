// knnf_select.h -- the bisections by which a full candidate buffer is cut down (used
// by the filter kernels' tighten).  Counting is the caller's: count(t) is the number
// of candidates at or below t.  Loop bounds and midpoints are unsigned: they span the
// whole range of distance bits and of linear indices.
#pragma once

#include <stdint.h>

namespace knnf {

// A distance bound t <= hi with at least K candidates at or below it, given that hi
// has: the first one found with at most `few`, else the smallest one above 0 (which is
// not counted).  n: its count (left alone where hi itself is returned, uncounted).
template <class Count>
__device__ __forceinline__ uint32_t cut_distance(uint32_t hi, int K, int few, int& n, Count count) {
    uint32_t lo = 0;  // fewer than K at lo (or lo = 0, not counted)
    // the K-th is rarely below an eighth of the bound
    if (hi > (3u << 23) && count(hi - (3u << 23)) < K) lo = hi - (3u << 23);
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        const int c = count(mid);
        if (c < K) {
            lo = mid;
        } else {
            hi = mid;
            n = c;
            if (c <= few) break;
        }
    }
    return hi;
}

// An index bound below which at least K and at most few >= K candidates lie: count(i)
// is the number of those with a smaller distance, fewer than K, and those of one
// distance with an index below i.  Indices are at most 2^31 - 2 and no two alike, so an
// index more is at most one candidate more, and the bound exists.
template <class Count>
__device__ __forceinline__ uint32_t cut_index(int K, int few, int& n, Count count) {
    uint32_t il = 0, ih = 0x80000000u;  // fewer than K below il, at least K below ih
    while (ih - il > 1) {
        const uint32_t mid = il + (ih - il) / 2;
        const int c = count(mid);
        if (c < K) {
            il = mid;
        } else {
            ih = mid;
            n = c;
            if (c <= few) break;
        }
    }
    return ih;
}

}  // namespace knnf
