// Formats of the forest data the host builds and the kernels read, the
// LDS-staged tree records above all.  No HIP headers, so the
// host-side builders (host_forest.cpp) also compile as plain C++.
#pragma once

#include <stdint.h>

#if defined(__HIP__) || defined(__HIPCC__)
#define TL_HOST_DEVICE __host__ __device__
#else
#define TL_HOST_DEVICE
#endif

namespace tl {

constexpr int kMaxRecordDepth = 11;

// The tree records that the kernels stage into LDS hold ranks instead of
// thresholds.  Trees are cut into groups of group_trees consecutive trees;
// within a group and for each feature, the distinct thresholds in ascending
// order are a dictionary c[0 .. n-1], n <= kMaxRank, and
//   rank(x) = how many of them are <= x   (n for a NaN x),
// so that x < c[i] iff rank(x) < i + 1 = the key of a node with threshold
// c[i] (key 0 for a NaN threshold, which no x is below).  A row is then two
// words, KV rank | batch rank << 16 and frequency rank | engine rank << 16,
// and one byte permute picks any of the four out of them.
//
// One record (byte ranges):
//   [4, 4 * 2^d)          node k (heap order from 1; children 2k, 2k + 1):
//                         key << 16 | selector, the selector's two bytes being
//                         the byte indices of the tested feature among the
//                         row's eight (frequency / engine size 0..3, KV /
//                         batch 4..7).  A row goes to 2k iff rank < key.
//   [4 * 2^d, 8 * 2^d)    value of leaf L, in word 2^d + L: where a walk
//                         that started at word 1 ends
//   [8 * 2^d, 16 * 2^d)   leaf boxes, 8 bytes per leaf: the lowest and the
//                         highest (KV rank | batch rank << 16) that the leaf's
//                         path allows (kEmptyBox for leaves no row reaches)
// A block of consecutive trees is one contiguous byte range, staged as is.
constexpr int32_t kMaxRank = 65534;
constexpr uint32_t kEmptyBoxLo = 0xffffffffu, kEmptyBoxHi = 0u;

TL_HOST_DEVICE inline uint32_t rank_record_bytes(int32_t depth) { return 16u << depth; }

// One feature's dictionary in one group, with a table of nb uniform buckets
// over its finite range: starts[b] = how many entries lie in buckets below b
// (nb + 1 of them).  The bucket of x is monotone in x, so an entry in a lower
// bucket than x's is <= x and one in a higher bucket is > x: only the entries
// of x's own bucket are searched.
struct RankFeature {
    uint32_t dict, starts;   // first entries in the shared arrays
    int32_t n, nb;
    float base, scale;
};
struct RankGroup {
    RankFeature f[4];
};

TL_HOST_DEVICE inline int32_t rank_bucket(const RankFeature& d, float x) {
    float q = (x - d.base) * d.scale;
    q = q > 0.0f ? q : 0.0f;   // (a NaN product, from a zero scale, goes to bucket 0)
    const float top = (float)(d.nb - 1);
    q = q < top ? q : top;
    return (int32_t)q;
}

TL_HOST_DEVICE inline uint32_t rank_of(const RankFeature& d, const float* dict, const uint16_t* starts, float x) {
    if (d.n == 0) return 0;
    if (x != x) return (uint32_t)d.n;
    const int32_t b = rank_bucket(d, x);
    uint32_t lo = starts[d.starts + (uint32_t)b], hi = starts[d.starts + (uint32_t)b + 1u];
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (dict[d.dict + mid] <= x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

}  // namespace tl
