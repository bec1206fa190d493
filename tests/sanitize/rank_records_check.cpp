// Checks of the rank records (host_forest.cpp, record_format.h) on random
// ensembles with NaN / +-inf / signed-zero / clustered thresholds, meant to
// run under AddressSanitizer and UndefinedBehaviorSanitizer:
//   - rank_of equals a linear count of the dictionary entries <= x, for
//     thresholds, their neighbours and special values;
//   - a walk over a record with the row's ranks ends at the leaf that a plain
//     walk on the fp32 row reaches, and finds that leaf's value there;
//   - that leaf's box holds the row's (KV, batch) ranks, and another row with
//     the same frequency and engine size reaches the leaf iff its ranks lie in
//     the box;
//   - every group's features have at most kMaxRank entries, also where the
//     forest has to be cut into several groups.
// Exits 1 on the first failure; prints a checksum of the records.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>
#include <random>
#include <vector>

#include "host_forest.h"

namespace {

int fail(const char* what, long long a, long long b) {
    std::fprintf(stderr, "FAIL: %s (%lld, %lld)\n", what, a, b);
    return 1;
}

int64_t plain_walk(const uint8_t* ft, const float* th, int depth, const float* x) {
    int64_t k = 0;
    for (int l = 0; l < depth; ++l) k = (x[ft[k]] < th[k]) ? 2 * k + 1 : 2 * k + 2;
    return k - ((1ll << depth) - 1);
}

}  // namespace

int main() {
    std::mt19937_64 rnd(7);
    auto uni = [&]() { return (double)(rnd() >> 11) * (1.0 / 9007199254740992.0); };
    uint64_t hash = 1469598103934665603ull;
    for (int trial = 0; trial < 40; ++trial) {
        const bool large = trial == 39;   // more than kMaxRank thresholds per feature
        const int depth = large ? 10 : (int)(rnd() % (tl::kMaxRecordDepth + 1));
        const int nf = 3 + (int)(rnd() % 2);
        const int T = large ? 400 : 1 + (int)(rnd() % (depth >= 9 ? 3 : 12));
        const int64_t n_int = (1ll << depth) - 1, n_leaf = 1ll << depth;
        std::vector<uint8_t> feature((size_t)(T * n_int));
        std::vector<float> threshold(feature.size()), leaf((size_t)(T * n_leaf));
        const float lo[4] = {1000.f, 0.f, -30.f, 1.f}, hi[4] = {2000.f, 70000.f, 300.f, 8.f};
        const bool cluster = trial % 5 == 1;
        for (size_t i = 0; i < feature.size(); ++i) {
            const int f = (int)(rnd() % nf);
            feature[i] = (uint8_t)f;
            const double u = uni();
            float t = (float)(lo[f] + (hi[f] - lo[f]) * uni());
            if (cluster) t = lo[f] + (hi[f] - lo[f]) * (float)std::pow(uni(), 20.0);
            if (!large) {
                if (u < 0.03) t = NAN;
                else if (u < 0.05) t = INFINITY;
                else if (u < 0.07) t = -INFINITY;
                else if (u < 0.09) t = -0.0f;
                else if (u < 0.11) t = 0.0f;
                else if (u < 0.25) t = std::floor(t);
                else if (u < 0.27) t = (float)(uni() < 0.5 ? 3e38 : -3e38);
            }
            threshold[i] = t;
        }
        for (auto& v : leaf) v = (float)(uni() - 0.5);
        tl::host::RankForest R;
        tl::host::build_rank_records(T, depth, feature.data(), threshold.data(), leaf.data(), R);
        const uint32_t bytes = tl::rank_record_bytes(depth);
        if (R.records.size() != (size_t)T * bytes + 64) return fail("record size", trial, (long long)R.records.size());
        if (large && R.groups.size() < 2) return fail("expected several groups", trial, (long long)R.groups.size());
        if ((int64_t)R.groups.size() != (T + R.group_trees - 1) / R.group_trees) return fail("groups", trial, R.group_trees);
        for (const unsigned char c : R.records) hash = (hash ^ c) * 1099511628211ull;
        for (const auto& g : R.groups)
            for (int f = 0; f < 4; ++f) {
                const tl::RankFeature& d = g.f[f];
                if (d.n > tl::kMaxRank) return fail("too many entries", trial, d.n);
                std::vector<float> probe = {NAN, INFINITY, -INFINITY, 0.f, -0.f, 1e30f, -1e30f,
                                            std::numeric_limits<float>::denorm_min(), 3.4e38f, -3.4e38f};
                for (int q = 0; q < 40; ++q) probe.push_back((float)(lo[f] + (hi[f] - lo[f]) * (1.2 * uni() - 0.1)));
                for (int q = 0; q < 40 && d.n > 0; ++q) {
                    const float c = R.dict[d.dict + rnd() % d.n];
                    probe.push_back(c);
                    probe.push_back(std::nextafter(c, INFINITY));
                    probe.push_back(std::nextafter(c, -INFINITY));
                }
                for (const float x : probe) {
                    uint32_t n = 0;
                    for (int32_t i = 0; i < d.n; ++i) n += std::isnan(x) || R.dict[d.dict + i] <= x;
                    if (tl::rank_of(d, R.dict.data(), R.starts.data(), x) != n) return fail("rank", trial, f);
                }
            }
        for (int t = 0; t < T; t += large ? 37 : 1) {
            const tl::RankGroup& g = R.groups[(size_t)(t / R.group_trees)];
            const uint32_t* w = (const uint32_t*)(R.records.data() + (size_t)t * bytes);
            auto rank = [&](int f, float x) { return tl::rank_of(g.f[f], R.dict.data(), R.starts.data(), x); };
            auto in = [&](int64_t L, const float* x) {
                const uint32_t lo_ = w[2 * n_leaf + 2 * L], hi_ = w[2 * n_leaf + 2 * L + 1];
                const uint32_t k = rank(1, x[1]), b = rank(2, x[2]);
                // as the kernels test it: clamped by hi, then lo
                const uint32_t ck = std::max(std::min(k, hi_ & 0xffffu), lo_ & 0xffffu);
                const uint32_t cb = std::max(std::min(b, hi_ >> 16), lo_ >> 16);
                return ck == k && cb == b;
            };
            for (int q = 0; q < 120; ++q) {
                float x[4];
                for (int f = 0; f < 4; ++f) {
                    x[f] = (float)(lo[f] + (hi[f] - lo[f]) * uni());
                    if (q % 3 == 0) x[f] = std::floor(x[f]);
                    if (q % 17 == 16 && rnd() % 3 == 0) x[f] = rnd() % 2 ? NAN : (rnd() % 2 ? INFINITY : -INFINITY);
                }
                const uint8_t* ft = feature.data() + t * n_int;
                const float* th = threshold.data() + t * n_int;
                const int64_t L = plain_walk(ft, th, depth, x);
                const uint32_t r[4] = {rank(0, x[0]), rank(1, x[1]), rank(2, x[2]), rank(3, x[3])};
                // the row's eight bytes: frequency, engine size, KV, batch
                const uint32_t lohi[2] = {r[0] | r[3] << 16, r[1] | r[2] << 16};
                unsigned char byte[8];
                std::memcpy(byte, lohi, 8);
                uint32_t k = 1;
                for (int l = 0; l < depth; ++l) {
                    const uint32_t v = byte[w[k] & 7u] | (uint32_t)byte[(w[k] >> 8) & 7u] << 8;
                    k = 2 * k + (v < (w[k] >> 16) ? 0 : 1);
                }
                if ((int64_t)k - n_leaf != L) return fail("walk", trial, t);
                if (std::memcmp(&w[k], &leaf[(size_t)(t * n_leaf + L)], 4) != 0) return fail("leaf value", trial, t);
                bool nan = false;
                for (int f = 0; f < 4; ++f) nan |= std::isnan(x[f]);
                if (nan) continue;
                if (!in(L, x)) return fail("row outside its leaf's box", trial, t);
                float y[4] = {x[0], x[1], x[2], x[3]};
                for (int m = 0; m < 6; ++m) {
                    y[1] = (float)std::floor(x[1] + (uni() - 0.5) * 3000.0);
                    y[2] = (float)std::floor(x[2] + (uni() - 0.5) * 20.0);
                    if (in(L, y) != (plain_walk(ft, th, depth, y) == L)) return fail("box", trial, t);
                }
            }
        }
    }
    std::printf("rank records ok checksum=%016llx\n", (unsigned long long)hash);
    return 0;
}
