// Host-side preparation of a tree ensemble (see host_forest.h).
#include "host_forest.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace tl {
namespace host {

// Going to 2k+1 means x < thr (an upper bound); going to 2k+2 means
// !(x < thr), i.e. x >= thr for non-NaN x (a lower bound).  A NaN threshold
// sends every row to 2k+2: no constraint there, and nothing reaches the 2k+1
// side, whose leaves get an empty box.
void leaf_boxes(int32_t n_trees, int32_t depth, const uint8_t* feature, const float* threshold,
                std::vector<Box>& out) {
    const int64_t n_int = (1ll << depth) - 1;
    const int64_t n_leaf = 1ll << depth;
    out.assign((size_t)(n_trees * n_leaf), Box{0, 0, 0, 0});
    for (int64_t t = 0; t < n_trees; ++t) {
        const uint8_t* ft = feature + t * n_int;
        const float* th = threshold + t * n_int;
        for (int64_t L = 0; L < n_leaf; ++L) {
            float lo[2] = {-INFINITY, -INFINITY}, hi[2] = {INFINITY, INFINITY};
            bool empty = false;
            int64_t k = 0;
            for (int32_t l = 0; l < depth; ++l) {
                const int bit = (int)((L >> (depth - 1 - l)) & 1);   // 0: to 2k+1, 1: to 2k+2
                const float thr = th[k];
                const int f = ft[k];
                if (bit == 0) {
                    if (std::isnan(thr)) empty = true;
                    else if (f == 1 || f == 2) hi[f - 1] = std::fmin(hi[f - 1], thr);
                } else if (!std::isnan(thr) && (f == 1 || f == 2)) {
                    lo[f - 1] = std::fmax(lo[f - 1], thr);
                }
                k = 2 * k + 1 + bit;
            }
            out[(size_t)(t * n_leaf + L)] = empty ? Box{INFINITY, -INFINITY, INFINITY, -INFINITY}
                                                  : Box{lo[0], hi[0], lo[1], hi[1]};
        }
    }
}

namespace {

// the order of non-NaN floats as the order of their 32-bit keys
uint32_t order_key(float x) {
    uint32_t b;
    std::memcpy(&b, &x, 4);
    if (b == 0x80000000u) b = 0;   // -0 compares equal to +0
    return (b & 0x80000000u) ? ~b : b | 0x80000000u;
}

// (key, node) pairs by key, least significant byte first; the pairs are
// (key << 32 | node)
void radix_sort(std::vector<uint64_t>& a, std::vector<uint64_t>& tmp) {
    tmp.resize(a.size());
    for (int shift = 32; shift < 64; shift += 11) {
        size_t count[2049] = {0};
        for (const uint64_t v : a) ++count[((v >> shift) & 2047u) + 1];
        if (count[((a.empty() ? 0 : a[0]) >> shift & 2047u) + 1] == a.size()) continue;   // one digit: nothing moves
        for (int i = 0; i < 2048; ++i) count[i + 1] += count[i];
        for (const uint64_t v : a) tmp[count[(v >> shift) & 2047u]++] = v;
        a.swap(tmp);
    }
}

// One feature's dictionary and bucket table from its nodes' (key, node)
// pairs; writes each node's rank key.
RankFeature build_feature(std::vector<uint64_t>& pairs, std::vector<uint64_t>& tmp, const float* threshold,
                          std::vector<float>& dict, std::vector<uint16_t>& starts, uint16_t* keys) {
    RankFeature d{};
    d.dict = (uint32_t)dict.size();
    d.starts = (uint32_t)starts.size();
    radix_sort(pairs, tmp);
    for (size_t i = 0; i < pairs.size(); ++i) {
        if (i == 0 || (pairs[i] >> 32) != (pairs[i - 1] >> 32)) {
            dict.push_back(threshold[(uint32_t)pairs[i]]);
            ++d.n;
        }
        keys[(uint32_t)pairs[i]] = (uint16_t)d.n;
    }
    // twice as many buckets as entries: most hold none or one
    d.nb = 1;
    while (d.nb < 2 * d.n && d.nb < (1 << 16)) d.nb *= 2;
    float lo = 0.0f, hi = 0.0f;
    bool any = false;
    for (int32_t i = 0; i < d.n; ++i) {
        const float x = dict[d.dict + i];
        if (!std::isfinite(x)) continue;
        if (!any) lo = x;
        hi = x;
        any = true;
    }
    d.base = lo;
    d.scale = hi > lo ? (float)((double)d.nb / ((double)hi - (double)lo)) : 0.0f;
    if (!std::isfinite(d.scale)) d.scale = 0.0f;
    int32_t i = 0;
    for (int32_t b = 0; b <= d.nb; ++b) {
        while (i < d.n && rank_bucket(d, dict[d.dict + i]) < b) ++i;
        starts.push_back((uint16_t)i);
    }
    return d;
}

}  // namespace

void build_rank_records(int32_t n_trees, int32_t depth, const uint8_t* feature, const float* threshold,
                        const float* leaf, RankForest& out) {
    const int64_t n_int = (1ll << depth) - 1;
    const int64_t n_leaf = 1ll << depth;
    out = RankForest();
    if (n_trees == 0) return;
    // the fewest groups of equal size whose features all have at most
    // kMaxRank nodes
    std::vector<uint32_t> nodes((size_t)n_trees * 4, 0);
    for (int64_t t = 0; t < n_trees; ++t)
        for (int64_t k = 0; k < n_int; ++k) ++nodes[(size_t)t * 4 + (feature[t * n_int + k] & 3)];
    int32_t per = n_trees;
    for (int32_t n_groups = 1;; ++n_groups) {
        per = (n_trees + n_groups - 1) / n_groups;
        bool fits = true;
        for (int32_t t0 = 0; t0 < n_trees && fits; t0 += per) {
            uint64_t sum[4] = {0, 0, 0, 0};
            for (int32_t t = t0; t < std::min(n_trees, t0 + per); ++t)
                for (int f = 0; f < 4; ++f) sum[f] += nodes[(size_t)t * 4 + f];
            for (int f = 0; f < 4; ++f) fits &= sum[f] <= (uint64_t)kMaxRank;
        }
        if (fits || per == 1) break;
    }
    out.group_trees = per;
    const uint32_t bytes = rank_record_bytes(depth);
    out.records.assign((size_t)n_trees * bytes + 64, 0);
    std::vector<uint16_t> keys;
    std::vector<uint64_t> pairs[4], tmp;
    struct Bounds {
        uint16_t lo[2], hi[2];
        bool empty;
    };
    std::vector<Bounds> at((size_t)2 * n_leaf);
    for (int32_t t0 = 0; t0 < n_trees; t0 += per) {
        const int32_t cnt = std::min(per, n_trees - t0);
        const uint8_t* ft = feature + t0 * n_int;
        const float* th = threshold + t0 * n_int;
        keys.assign((size_t)(cnt * n_int), 0);   // (0: a NaN threshold)
        for (auto& p : pairs) p.clear();
        for (int64_t i = 0; i < cnt * n_int; ++i)
            if (!std::isnan(th[i])) pairs[ft[i] & 3].push_back((uint64_t)order_key(th[i]) << 32 | (uint64_t)i);
        RankGroup g;
        for (int f = 0; f < 4; ++f) g.f[f] = build_feature(pairs[f], tmp, th, out.dict, out.starts, keys.data());
        out.groups.push_back(g);
        for (int32_t t = 0; t < cnt; ++t) {
            unsigned char* rec = out.records.data() + (size_t)(t0 + t) * bytes;
            uint32_t* word = (uint32_t*)rec;
            at[1] = Bounds{{0, 0}, {0xffff, 0xffff}, false};
            for (int64_t k = 1; k <= n_int; ++k) {
                const int f = ft[t * n_int + k - 1] & 3;
                const uint32_t key = keys[(size_t)(t * n_int + k - 1)];
                // bytes of the row pair: frequency 0-1, engine size 2-3, KV 4-5, batch 6-7
                const uint32_t first = f == 0 ? 0u : f == 1 ? 4u : f == 2 ? 6u : 2u;
                word[k] = key << 16 | (first + 1) << 8 | first;
                Bounds l = at[(size_t)k], r = at[(size_t)k];
                if (f == 1 || f == 2) {
                    if (key == 0) l.empty = true;
                    else l.hi[f - 1] = std::min<uint16_t>(l.hi[f - 1], (uint16_t)(key - 1));
                    r.lo[f - 1] = std::max<uint16_t>(r.lo[f - 1], (uint16_t)key);
                }
                at[(size_t)(2 * k)] = l;
                at[(size_t)(2 * k + 1)] = r;
            }
            std::memcpy(rec + 4 * n_leaf, leaf + (t0 + t) * n_leaf, 4 * (size_t)n_leaf);
            uint32_t* box = (uint32_t*)(rec + 8 * n_leaf);
            for (int64_t L = 0; L < n_leaf; ++L) {
                const Bounds& b = at[(size_t)(n_leaf + L)];
                const bool none = b.empty || b.lo[0] > b.hi[0] || b.lo[1] > b.hi[1];
                box[2 * L] = none ? kEmptyBoxLo : (uint32_t)b.lo[1] << 16 | b.lo[0];
                box[2 * L + 1] = none ? kEmptyBoxHi : (uint32_t)b.hi[1] << 16 | b.hi[0];
            }
        }
    }
}

}  // namespace host
}  // namespace tl
