// Host-side preparation of a tree ensemble for the kernels (plain C++, no
// HIP): the KV / batch box of every leaf for trees too deep to stage, the rank
// records of the others.  Trees are complete, depth d, heap order: internal node k tests x[feature] < threshold and continues at
// 2k+1 if true, at 2k+2 otherwise (Sec. 4.3.1 model M).
#pragma once

#include <stdint.h>

#include <vector>

#include "record_format.h"

namespace tl {
namespace host {

// The bounds a leaf's root-to-leaf path puts on features 1 (KV) and 2
// (batch) as half-open intervals: a row with kv_lo <= KV < kv_hi and
// batch_lo <= batch < batch_hi reaches the leaf whenever a row with the same
// frequency and engine size does.  Empty (lo = +inf, hi = -inf) for leaves
// no row can reach.
struct Box {
    float kv_lo, kv_hi, batch_lo, batch_hi;
};

// boxes of every leaf of every tree, [n_trees][2^depth]
void leaf_boxes(int32_t n_trees, int32_t depth, const uint8_t* feature, const float* threshold,
                std::vector<Box>& out);

// The rank records of all trees (rank_record_bytes(depth) each, back to back,
// plus 64 bytes of padding), and the groups, dictionaries and bucket tables
// that rank rows for them (record_format.h).  depth <= kMaxRecordDepth,
// n_features 3 or 4.
struct RankForest {
    int32_t group_trees = 0;                // every group but the last has this many trees
    std::vector<RankGroup> groups;
    std::vector<float> dict;
    std::vector<uint16_t> starts;
    std::vector<unsigned char> records;
};
void build_rank_records(int32_t n_trees, int32_t depth, const uint8_t* feature, const float* threshold,
                        const float* leaf, RankForest& out);

}  // namespace host
}  // namespace tl
