// The model M (Sec. 4.3.1) at one frequency per scenario on the projection
// grid: out[s][j] = M(f_s, KV[s][j], B[s][j] [, E_s]), f_s = freqs[fidx[s]]
// (scenarios with fidx[s] < 0 are skipped) or one frequency for all.  This is the query of
// the admission checks (Sec. 4.3.2 check 2 asks M at the maximum frequency
// for every projected iteration) and of one probe of a search over
// frequencies (Sec. 4.5).
//
// A wavefront takes RPL (1 or 2) stripes of 64 consecutive iterations of one
// scenario, RPL rows per lane; the rows differ, so every lane walks every tree (the grid
// kernel's leaf reuse needs many frequencies on the same row sequence).
// Sixteen wavefronts of a workgroup share two LDS buffers of tree-record
// blocks, copied straight from global memory and handed over without block
// barriers (stage_acquire / stage_release, which also set the wavefronts'
// issue priorities).  A lane walks its RPL rows through up to four trees at
// once, so RPL x trees chains of dependent LDS reads overlap (deep trees leave
// room for only two trees per block).  Leaves are added as an fp32 running sum
// in tree order, as everywhere in the library.
//
// On horizons of at least 64 x RPL iterations and grids of at least one
// workgroup per CU, forest_column_reuse_kernel gives each lane RPL (16, else
// 8) consecutive iterations instead and reuses leaves along them: every lane
// walks its first and last row, and the rows in between take those leaves
// where their boxes hold them (the grid kernel's box test, per lane).
//
// Forests too deep for LDS records are walked from global memory.
//
// Rows mode (P.rows): the same kernel on arbitrary feature rows, lane l of
// item i taking rows i*64*RPL + l + 64 r; every row carries its own
// frequency and engine size.  tl_forest_predict uses it for 3- and
// 4-feature forests with LDS records.
#include <algorithm>

#include "device_util.h"
#include "tl_internal.h"
#include "forest_walk.h"

namespace tl {
namespace {

constexpr int kColWaves = 16;
constexpr int kColThreads = kColWaves * kWave;
constexpr size_t kColLdsBudget = 152 * 1024;
constexpr size_t kColLdsHalf = 76 * 1024;

template <int RPL>
struct ColumnItem {
    int64_t s;
    int32_t j[RPL];     // this lane's iterations (clamped into the horizon)
    bool row[RPL];      // ... and whether each is inside it
    bool valid;         // the wavefront has a scenario
};

template <int RPL>
__device__ __forceinline__ ColumnItem<RPL> column_item(const ColumnParams& P, int64_t item) {
    const int32_t span = kWave * RPL;
    const int32_t n_cols = (P.H + span - 1) / span;
    ColumnItem<RPL> c;
    c.valid = item < P.S * n_cols;
    c.s = c.valid ? item / n_cols : 0;
    // a scenario without a frequency to evaluate (index < 0) is skipped
    if (P.fidx && P.fidx[c.s] < 0) c.valid = false;
    const int32_t j0 = (int32_t)(item % n_cols) * span + lane_id();
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int32_t j = j0 + r * kWave;
        c.row[r] = c.valid && j < P.H;
        c.j[r] = min(j, P.H - 1);
    }
    return c;
}

__device__ __forceinline__ float column_freq(const ColumnParams& P, int64_t s) {
    return P.fidx ? P.freqs[max(P.fidx[s], 0)] : P.freq;
}

// Walks NT consecutive staged trees for the RPL rows of a lane and adds the
// leaves to each row's sum in tree order.
template <int NT, int RPL>
__device__ __forceinline__ void add_leaves(uint32_t tree, uint32_t rec_bytes, int32_t depth,
                                           const uint32_t (&row)[RPL], const uint32_t (&fe)[RPL], float (&acc)[RPL]) {
    uint32_t k[RPL][NT];
    walk_rows<NT, RPL>(tree, rec_bytes, depth, row, fe, k);
#pragma unroll
    for (int r = 0; r < RPL; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r] += leaf_value(k[r][t]);
}

template <int NF, int RPL, bool ROWS>
__global__ __launch_bounds__(kColThreads) void forest_column_lds_kernel(RankDev D, TreeBlocks B, ColumnParams P) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t rec_bytes = staged_bytes<true>(D.depth);
    const uint32_t buf_bytes = stage_buffer_bytes(B.tb, rec_bytes);
    const int wave = threadIdx.x / kWave;
    const int64_t item = __builtin_amdgcn_readfirstlane((int64_t)blockIdx.x * kColWaves + wave);
    StageSync* sync = (StageSync*)(smem + 2 * buf_bytes);
    if (threadIdx.x == 0) stage_sync_init(sync);
    if (B.n_blocks > 0) stage_block<true>(D, B, 0, lds_addr(smem), wave, kColWaves);
    float acc[RPL];
    int64_t o[RPL];     // output index of each row, < 0: none
    int64_t in[RPL];    // input index of each row
    bool valid;         // the wavefront has rows (uniform)
    int64_t s = 0;
    if (ROWS) {
        const int64_t first = item * (kWave * RPL);
        valid = first < P.n_rows;
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int64_t i = first + lane_id() + r * kWave;
            o[r] = i < P.n_rows ? i : -1;
            in[r] = valid ? min(i, P.n_rows - 1) : 0;
        }
    } else {
        const ColumnItem<RPL> c = column_item<RPL>(P, item);
        valid = c.valid;
        s = c.s;
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            in[r] = c.s * P.H + c.j[r];
            o[r] = c.row[r] ? in[r] : -1;
        }
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) acc[r] = D.base;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    bool sync_ok = true;
    for (int32_t grp = 0; grp < D.n_groups; ++grp) {
        // this group's ranks of the rows
        uint32_t row[RPL], fe[RPL];
        if (valid) {
            const uint32_t fe_s = ROWS ? 0u : rank_lane(D, grp, column_freq(P, s), NF == 4 ? P.engine[s] : 0.0f);
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                if (ROWS) {
                    const float* x = P.rows + in[r] * NF;
                    row[r] = rank_row(D, grp, x[1], x[2]);
                    fe[r] = rank_lane(D, grp, x[0], NF == 4 ? x[3] : 0.0f);
                } else {
                    row[r] = rank_row(D, grp, (float)P.kv[in[r]], (float)P.batch[in[r]]);
                    fe[r] = fe_s;
                }
                // the ranks are complete before this wavefront stages again
                asm volatile("" ::"v"(row[r]), "v"(fe[r]));
            }
        }
        const int32_t b_end = min((grp + 1) * B.group_blocks, B.n_blocks);
        for (int32_t b = grp * B.group_blocks; b < b_end; ++b) {
            const uint32_t buf = lds_addr(smem) + (uint32_t)(b & 1) * buf_bytes;
            if (b > 0) sync_ok &= stage_acquire<2, true>(sync, b, kColWaves, D, B, buf);
            if (valid) {
                const int32_t cnt = block_count(D, B, b, block_first(D, B, b));
                int32_t t = 0;
                for (; t + 4 <= cnt; t += 4)
                    add_leaves<4, RPL>(buf + t * rec_bytes, rec_bytes, D.depth, row, fe, acc);
                for (; t + 2 <= cnt; t += 2)
                    add_leaves<2, RPL>(buf + t * rec_bytes, rec_bytes, D.depth, row, fe, acc);
                if (t < cnt) add_leaves<1, RPL>(buf + t * rec_bytes, rec_bytes, D.depth, row, fe, acc);
            }
            stage_release(sync, b, kColWaves);
        }
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r)
        if (o[r] >= 0) P.out[o[r]] = sync_ok ? acc[r] : __builtin_nanf("");
}

// Leaf reuse along a lane's RPL consecutive rows with two anchors: every lane
// walks its first and last row through NT (1 or 2) consecutive staged trees in
// one interleaved pass (full wavefronts), keeps those leaves' values and KV /
// batch boxes, and gives every row in between the value of an anchor leaf
// whose box holds it (the frequency and engine size are the scenario's, so a
// row inside a leaf's box reaches that leaf), or of the leaf of the lane's
// last walk in between.  Only rows in none of these boxes walk, the trees
// they need, both in one pass when the wavefront needs both.
template <int NT, int RPL>
__device__ __forceinline__ void add_leaves_anchored(uint32_t tree, uint32_t rec_bytes, int32_t depth, uint32_t fe,
                                                    const uint32_t (&row)[RPL], float (&acc)[RPL]) {
    float va[2][NT];
    Box ba[2][NT];
    {
        const uint32_t rows[2] = {row[0], row[RPL - 1]}, fes[2] = {fe, fe};
        uint32_t ka[2][NT];
        walk_rows<NT, 2>(tree, rec_bytes, depth, rows, fes, ka);
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                va[e][t] = leaf_value(ka[e][t]);
                ba[e][t] = leaf_box(ka[e][t], tree + t * rec_bytes);
            }
    }
    float vl[NT];
    Box bl[NT];   // the last walk's leaf (none yet: empty box)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        vl[t] = 0.0f;
        bl[t] = empty_box();
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        float v[NT];
        if (r == 0 || r == RPL - 1) {
#pragma unroll
            for (int t = 0; t < NT; ++t) v[t] = va[r == 0 ? 0 : 1][t];
        } else {
            bool need[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bool in0 = in_box(ba[0][t], row[r]);
                const bool in1 = in_box(ba[1][t], row[r]);
                need[t] = !in0 && !in1 && !in_box(bl[t], row[r]);
                v[t] = in0 ? va[0][t] : (in1 ? va[1][t] : vl[t]);
            }
            if (NT == 2 && __builtin_amdgcn_ballot_w64(need[0]) != 0 &&
                __builtin_amdgcn_ballot_w64(need[NT - 1]) != 0) {
                uint32_t k[NT];
                walk<NT>(tree, rec_bytes, depth, row[r], fe, k);
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (need[t]) {
                        v[t] = vl[t] = leaf_value(k[t]);
                        bl[t] = leaf_box(k[t], tree + t * rec_bytes);
                    }
            } else {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (need[t]) {
                        uint32_t k[1];
                        walk<1>(tree + t * rec_bytes, rec_bytes, depth, row[r], fe, k);
                        v[t] = vl[t] = leaf_value(k[0]);
                        bl[t] = leaf_box(k[0], tree + t * rec_bytes);
                    }
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r] += v[t];
        asm volatile("" ::"v"(acc[r]));
    }
}

// M at one frequency per scenario with leaf reuse along each lane's RPL
// consecutive iterations (a wavefront takes 64 x RPL consecutive
// iterations of one scenario); staging as in forest_column_lds_kernel.
// LIVE: the items are the first *P.n_live entries of P.order.
template <int RPL, bool LIVE>
__global__ __launch_bounds__(kColThreads) void forest_column_reuse_kernel(RankDev D, TreeBlocks B, ColumnParams P) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t rec_bytes = rank_record_bytes(D.depth);
    const uint32_t buf_bytes = stage_buffer_bytes(B.tb, rec_bytes);
    const int wave = threadIdx.x / kWave;
    const int64_t item = __builtin_amdgcn_readfirstlane((int64_t)blockIdx.x * kColWaves + wave);
    const int32_t span = kWave * RPL;
    const int32_t n_cols = (P.H + span - 1) / span;
    const int64_t n_items = LIVE ? (int64_t)*P.n_live : P.S * n_cols;
    // a workgroup wholly past the live items has nothing to stage for
    if (LIVE && (int64_t)blockIdx.x * kColWaves >= n_items) return;
    bool valid = item < n_items;
    // the (scenario, column) pair: item itself, or its entry of the work order
    const int64_t code = !valid ? 0 : P.order ? (int64_t)P.order[item] : item;
    const int64_t s = code / n_cols;
    if (P.fidx && P.fidx[s] < 0) valid = false;
    const int32_t j0 = (int32_t)(code % n_cols) * span + lane_id() * RPL;
    float acc[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) acc[r] = D.base;
    StageSync* sync = (StageSync*)(smem + 2 * buf_bytes);
    if (threadIdx.x == 0) stage_sync_init(sync);
    if (B.n_blocks > 0) stage_block(D, B, 0, lds_addr(smem), wave, kColWaves);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    bool sync_ok = true;
    for (int32_t grp = 0; grp < D.n_groups; ++grp) {
        uint32_t row[RPL], fe = 0;
        if (valid) {
            fe = rank_lane(D, grp, column_freq(P, s), P.engine ? P.engine[s] : 0.0f);
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int64_t i = s * P.H + min(j0 + r, P.H - 1);
                row[r] = rank_row(D, grp, (float)P.kv[i], (float)P.batch[i]);
                // the ranks are complete before this wavefront stages again
                asm volatile("" ::"v"(row[r]));
            }
            asm volatile("" ::"v"(fe));
        }
        const int32_t b_end = min((grp + 1) * B.group_blocks, B.n_blocks);
        for (int32_t b = grp * B.group_blocks; b < b_end; ++b) {
            const uint32_t buf = lds_addr(smem) + (uint32_t)(b & 1) * buf_bytes;
            if (b > 0) sync_ok &= stage_acquire(sync, b, kColWaves, D, B, buf);
            if (valid) {
                const int32_t cnt = block_count(D, B, b, block_first(D, B, b));
                int32_t t = 0;
                for (; t + 2 <= cnt; t += 2)
                    add_leaves_anchored<2, RPL>(buf + t * rec_bytes, rec_bytes, D.depth, fe, row, acc);
                if (t < cnt) add_leaves_anchored<1, RPL>(buf + t * rec_bytes, rec_bytes, D.depth, fe, row, acc);
            }
            stage_release(sync, b, kColWaves);
        }
    }
    if (valid) {
#pragma unroll
        for (int r = 0; r < RPL; ++r)
            if (j0 + r < P.H) P.out[s * P.H + j0 + r] = sync_ok ? acc[r] : __builtin_nanf("");
    }
}

// Global-memory walks for forests without LDS records.
template <int NF>
__global__ __launch_bounds__(256) void forest_column_global_kernel(const uint2* __restrict__ nodes,
                                                                  const float* __restrict__ leaves,
                                                                  int32_t n_trees, int32_t depth, float base,
                                                                  ColumnParams P) {
    const int64_t item = (int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    const ColumnItem<1> c = column_item<1>(P, item);
    if (!c.row[0]) return;
    float x[4];
    x[0] = column_freq(P, c.s);
    x[1] = (float)P.kv[c.s * P.H + c.j[0]];
    x[2] = (float)P.batch[c.s * P.H + c.j[0]];
    x[3] = NF == 4 ? P.engine[c.s] : 0.0f;
    const int64_t stride = (int64_t)1 << depth;
    const int32_t n_int = (1 << depth) - 1;
    float acc = base;
    for (int32_t t = 0; t < n_trees; ++t) {
        const uint2* nd = nodes + t * stride;
        int32_t k = 0;
        for (int32_t level = 0; level < depth; ++level) {
            const uint2 w = nd[k];
            const float v = x[w.y & 3u];
            k = 2 * k + (v < __uint_as_float(w.x) ? 1 : 2);
        }
        acc += leaves[t * stride + (k - n_int)];
    }
    P.out[c.s * P.H + c.j[0]] = acc;
}

// Trees per staged block: double buffers within the LDS budget.  HALF: of
// trees without their boxes.
template <bool HALF>
int32_t column_trees_per_block(const ForestDev& f, size_t budget, size_t* lds) {
    if (!f.records || f.n_trees == 0) return 0;
    const uint32_t rec_bytes = staged_bytes<HALF>(f.depth);
    // two tree buffers and their hand-over counters
    auto bytes = [&](int32_t n) { return 2 * (size_t)stage_buffer_bytes(n, rec_bytes) + sizeof(StageSync); };
    // whole quads of trees where four fit
    int32_t tb = 64;
    while (tb > 1 && bytes(tb) > budget) tb -= tb > 4 ? 4 : 1;
    if (bytes(tb) > budget) return 0;
    *lds = bytes(tb);
    return tb;
}

template <int NF, int RPL, bool ROWS = false>
hipError_t launch_column_lds(const ForestDev& f, const ColumnParams& c, hipStream_t stream) {
    const int64_t span = kWave * RPL;
    const int64_t items = ROWS ? (c.n_rows + span - 1) / span : c.S * ((c.H + span - 1) / span);
    // Half a CU's LDS where there are workgroups for both halves, all of it
    // where there are not: fewer, larger copies (500 trees of depth 8: 200 000
    // rows 182 us with all of it, 197 with half; a million 577 and 544).
    size_t lds = 0;
    const int32_t tb =
        column_trees_per_block<true>(f, items > (int64_t)kColWaves * f.cus ? kColLdsHalf : kColLdsBudget, &lds);
    const auto kern = forest_column_lds_kernel<NF, RPL, ROWS>;
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t blocks = (items + kColWaves - 1) / kColWaves;
    if (!grid_fits(blocks, kColThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kColThreads), lds, stream, rank_dev(f),
                       tree_blocks(f.n_trees, f.group_trees, tb), c);
    return hipGetLastError();
}

// Rows per lane of the leaf-reuse kernel for these rows: 16 (else 8) where
// the horizon fills a wavefront's 64 x RPL rows and the grid still gives
// every CU a workgroup; 0 when the kernel does not apply.
int reuse_rows_per_lane(const ForestDev& f, const ColumnParams& c) {
    size_t lds = 0;
    if (c.rows || column_trees_per_block<false>(f, kColLdsBudget, &lds) <= 0) return 0;
    for (int r : {16, 8}) {
        const int64_t items = c.S * ((c.H + kWave * r - 1) / (kWave * r));
        if (c.H >= kWave * r && items >= (int64_t)kColWaves * f.cus) return r;
    }
    return 0;
}

template <int RPL>
hipError_t launch_column_reuse(const ForestDev& f, const ColumnParams& c, int32_t tb, size_t lds,
                               hipStream_t stream) {
    const int64_t items = c.S * ((c.H + kWave * RPL - 1) / (kWave * RPL));
    const auto kern =
        c.n_live ? forest_column_reuse_kernel<RPL, true> : forest_column_reuse_kernel<RPL, false>;
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t blocks = (items + kColWaves - 1) / kColWaves;
    if (!grid_fits(blocks, kColThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kColThreads), lds, stream, rank_dev(f),
                       tree_blocks(f.n_trees, f.group_trees, tb), c);
    return hipGetLastError();
}

template <int NF>
hipError_t launch_column(const ForestDev& f, const ColumnParams& c, hipStream_t stream) {
    size_t lds = 0;
    const int32_t tb = column_trees_per_block<false>(f, kColLdsBudget, &lds);
    if (tb > 0) {
        const int rpl = reuse_rows_per_lane(f, c);
        if (rpl == 16) return launch_column_reuse<16>(f, c, tb, lds, stream);
        if (rpl == 8) return launch_column_reuse<8>(f, c, tb, lds, stream);
    }
    if (tb > 0) {
        // rows per lane: 2, with twice the chains to overlap, where that
        // leaves every CU a workgroup and no idle stripes on short horizons
        if (c.H > kWave && c.S * ((c.H + kWave * 2 - 1) / (kWave * 2)) >= (int64_t)kColWaves * f.cus)
            return launch_column_lds<NF, 2>(f, c, stream);
        return launch_column_lds<NF, 1>(f, c, stream);
    }
    const int64_t items = c.S * ((c.H + kWave - 1) / kWave);
    if (!grid_fits((items + 3) / 4, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(forest_column_global_kernel<NF>, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, stream,
                       f.nodes, f.leaves, f.n_trees, f.depth, f.base_score, c);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_forest_column(const ForestDev& f, const ColumnParams& c, hipStream_t stream) {
    if (c.S == 0) return hipSuccess;
    // More wavefronts of one row a lane than one launch takes: parts of whole
    // scenarios, in their own order.
    const int64_t most = std::max<int64_t>(1, (kMaxLaunchWaves - kColWaves) / ((c.H + kWave - 1) / kWave));
    if (c.S > kMaxParts * most) return hipErrorInvalidConfiguration;
    for (int64_t s0 = 0; s0 < c.S && c.S > most; s0 += most) {
        ColumnParams p = c;
        p.S = std::min(most, c.S - s0);
        p.kv += s0 * c.H;
        p.batch += s0 * c.H;
        if (p.fidx) p.fidx += s0;
        if (p.engine) p.engine += s0;
        p.out += s0 * c.H;
        p.order = nullptr;
        p.n_live = nullptr;
        const hipError_t e = launch_forest_column(f, p, stream);
        if (e != hipSuccess || s0 + most >= c.S) return e;
    }
    return f.n_features == 4 ? launch_column<4>(f, c, stream) : launch_column<3>(f, c, stream);
}

namespace {

__global__ void column_live_clear_kernel(int32_t* n_live) { *n_live = 0; }

// The live items of the leaf-reuse kernel: entry i of the work order (or
// item i) is kept when its scenario is selected (fidx >= 0); a wavefront's
// kept entries stay in order and take consecutive slots from one atomic add.
__global__ __launch_bounds__(256) void column_live_kernel(const uint32_t* __restrict__ order,
                                                          const int32_t* __restrict__ fidx, int64_t n_items,
                                                          int32_t n_cols, uint32_t* __restrict__ live,
                                                          int32_t* __restrict__ n_live) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t code = 0;
    bool keep = false;
    if (i < n_items) {
        code = order ? order[i] : (uint32_t)i;
        keep = fidx[code / (uint32_t)n_cols] >= 0;
    }
    const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
    if (m == 0) return;
    int32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(n_live, (int32_t)__builtin_popcountll(m));
    base = __shfl(base, 0);
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (keep) live[base + (int32_t)below] = code;
}

// The leaf-reuse kernel's work order for c's rows (p.n = 0: none).  It is
// only planned for grids of at least two workgroups per CU: with one, the
// kernel takes as long as its slowest wavefront whatever the order.
hipError_t plan_column_order(const ForestDev& f, const ColumnParams& c, int* rpl, PairOrderPlan* p) {
    *p = PairOrderPlan{0, 0, 0, 0};
    if (c.S == 0) return hipSuccess;
    *rpl = reuse_rows_per_lane(f, c);
    if (*rpl == 0) return hipSuccess;
    const int64_t span = kWave * *rpl;
    const int64_t items = c.S * ((c.H + span - 1) / span);
    return pair_order_plan(f, items, 2 * (int64_t)kColWaves * f.cus, p);
}

}  // namespace

hipError_t column_order_bytes(const ForestDev& f, const ColumnParams& c, size_t* bytes) {
    int rpl = 0;
    PairOrderPlan p;
    const hipError_t e = plan_column_order(f, c, &rpl, &p);
    *bytes = e == hipSuccess ? p.bytes : 0;
    return e;
}

hipError_t order_forest_column(const ForestDev& f, ColumnParams& c, void* ws, hipStream_t stream) {
    int rpl = 0;
    PairOrderPlan p;
    hipError_t e = plan_column_order(f, c, &rpl, &p);
    if (e != hipSuccess || p.n == 0) return e;
    return pair_order(f, p, c.kv, c.batch, c.H, kWave * rpl, ws, &c.order, stream);
}

hipError_t column_live_bytes(const ForestDev& f, const ColumnParams& c, size_t* bytes) {
    *bytes = 0;
    if (c.S == 0 || !c.fidx) return hipSuccess;
    const int rpl = reuse_rows_per_lane(f, c);
    if (rpl == 0) return hipSuccess;
    const int64_t span = kWave * rpl;
    const int64_t items = c.S * ((c.H + span - 1) / span);
    // as for the work order: with one workgroup per CU the launch lasts as
    // long as its slowest workgroup, compacted or not
    if (items < 2 * (int64_t)kColWaves * f.cus) return hipSuccess;
    *bytes = (((size_t)items * sizeof(uint32_t) + 255) & ~(size_t)255) + 256;
    return hipSuccess;
}

hipError_t launch_forest_column_live(const ForestDev& f, const ColumnParams& c, void* ws, hipStream_t stream) {
    const int rpl = ws && c.fidx && c.S > 0 ? reuse_rows_per_lane(f, c) : 0;
    if (rpl == 0) return launch_forest_column(f, c, stream);
    const int32_t span = kWave * rpl;
    const int32_t n_cols = (c.H + span - 1) / span;
    const int64_t items = c.S * n_cols;
    uint32_t* live = (uint32_t*)ws;
    int32_t* n_live = (int32_t*)((unsigned char*)ws + (((size_t)items * sizeof(uint32_t) + 255) & ~(size_t)255));
    hipLaunchKernelGGL(column_live_clear_kernel, dim3(1), dim3(1), 0, stream, n_live);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!grid_fits((items + 255) / 256, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(column_live_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream, c.order,
                       c.fidx, items, n_cols, live, n_live);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    ColumnParams d = c;
    d.order = live;
    d.n_live = n_live;
    return launch_forest_column(f, d, stream);
}

hipError_t launch_forest_rows_lds(const ForestDev& f, const float* rows, int64_t n_rows, float* out,
                                  hipStream_t stream) {
    size_t lds = 0;
    const int32_t tb = (f.n_features == 3 || f.n_features == 4) ? column_trees_per_block<false>(f, kColLdsBudget, &lds) : 0;
    if (tb <= 0) return hipErrorNotSupported;
    if (n_rows == 0) return hipSuccess;
    // Parts of as many rows as one launch takes at one a lane.
    const int64_t most = (kMaxLaunchWaves - kColWaves) * kWave;
    if (n_rows > kMaxParts * most) return hipErrorInvalidConfiguration;
    for (int64_t r0 = 0; n_rows > most && r0 < n_rows; r0 += most) {
        const hipError_t e =
            launch_forest_rows_lds(f, rows + r0 * f.n_features, std::min(most, n_rows - r0), out + r0, stream);
        if (e != hipSuccess || r0 + most >= n_rows) return e;
    }
    ColumnParams c{};
    c.rows = rows;
    c.n_rows = n_rows;
    c.out = out;
    const bool four = f.n_features == 4;
    // two rows a lane where that leaves every CU a workgroup (four, at half
    // the wavefronts a CU: 500 trees of depth 8 on 3 M rows 1559 against 1443 us,
    // 2000 of depth 10 on 1.5 M 6037 against 4793)
    if (n_rows >= (int64_t)2 * kColThreads * f.cus)
        return four ? launch_column_lds<4, 2, true>(f, c, stream) : launch_column_lds<3, 2, true>(f, c, stream);
    return four ? launch_column_lds<4, 1, true>(f, c, stream) : launch_column_lds<3, 1, true>(f, c, stream);
}

}  // namespace tl
