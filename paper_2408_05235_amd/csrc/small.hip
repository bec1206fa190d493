// The model M (Sec. 4.3.1) for calls with few rows, in two launches.
//
// The grid and column kernels give a wavefront whole runs of rows and every
// tree: what a large call needs, but a call with a few thousand rows then
// leaves nearly all CUs idle while a handful of wavefronts walk every tree in
// turn.  The ensemble's sum has a fixed order (an fp32 running sum in tree
// order), the walks have none, so a small call is cut along the trees too:
//
//   forest_leaves_kernel   a workgroup takes a tile of rows (one row a lane)
//       and a chunk of trees staged into LDS, and writes the value of the
//       leaf that each row reaches in each tree to a scratch array
//       [64 rows][tree][row of the 64].  Four trees are walked at once (four
//       chains of dependent LDS reads in flight a lane).
//   forest_sum_kernel      adds each row's values in tree order: eight
//       wavefronts fetch the values of 64 rows, 32 trees a wavefront in
//       flight, through LDS, and one of them adds.
//
// Rows are those of the projection grid, of one frequency per scenario, or a
// caller's own; row i's result is out[i] in each case.  Calls whose scratch
// would exceed kSmallScratchBytes run in slices of rows.
#include <algorithm>

#include "device_util.h"
#include "tl_internal.h"
#include "forest_walk.h"

namespace tl {
namespace {

enum RowKind { kGridRows, kColumnRows, kOwnRows };

struct SmallRow {
    float xf, kv, bs, xe;
    bool on;        // the row's result is wanted
};

template <RowKind KIND>
__device__ __forceinline__ SmallRow small_row(const SmallParams& P, int64_t i) {
    SmallRow r;
    if (KIND == kOwnRows) {
        const float* x = P.rows + i * P.nf;
        r.xf = x[0];
        r.kv = x[1];
        r.bs = x[2];
        r.xe = P.nf == 4 ? x[3] : 0.0f;
        r.on = true;
        return r;
    }
    const int64_t line = i / P.H;                       // scenario, or scenario * F + frequency
    const int64_t s = KIND == kGridRows ? line / P.F : line;
    const int64_t at = s * P.H + (i - line * P.H);
    const int32_t f = KIND == kGridRows ? (int32_t)(line - s * P.F) : P.fidx ? P.fidx[s] : 0;
    r.xf = KIND == kColumnRows && !P.fidx ? P.freq : P.freqs[max(f, 0)];
    r.kv = (float)P.kv[at];
    r.bs = (float)P.batch[at];
    r.xe = P.engine ? P.engine[s] : 0.0f;
    r.on = f >= 0;
    return r;
}

template <int NT>
__device__ __forceinline__ void put_leaves(uint32_t tree, uint32_t bytes, int32_t depth, uint32_t row, uint32_t fe,
                                           float* to, bool on) {
    uint32_t k[NT];
    walk<NT>(tree, bytes, depth, row, fe, k);
    float v[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) v[t] = leaf_value(k[t]);
    if (on) {
#pragma unroll
        for (int t = 0; t < NT; ++t) to[t * kWave] = v[t];
    }
}

// Workgroup (x, y): rows [first + x * 64 * WAVES, ...) and tree chunk y
// (C.tb trees), staged tb trees at a time into two buffers.
template <RowKind KIND, int WAVES>
__global__ __launch_bounds__(WAVES* kWave) void forest_leaves_kernel(RankDev D, TreeBlocks C, int32_t tb,
                                                                     SmallParams P, int64_t first_row,
                                                                     int64_t n_rows, float* __restrict__ values) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t bytes = staged_bytes<true>(D.depth);
    const uint32_t buf_bytes = stage_buffer_bytes(tb, bytes);
    const int wave = threadIdx.x / kWave;
    const int32_t chunk = (int32_t)blockIdx.y;
    const int32_t t0 = block_first(D, C, chunk), t1 = t0 + block_count(D, C, chunk, t0);
    stage_trees<true>(D, t0, min(tb, t1 - t0), lds_addr(smem), wave, WAVES);
    const int64_t r = (int64_t)blockIdx.x * (WAVES * kWave) + threadIdx.x;   // within the slice
    const SmallRow x = small_row<KIND>(P, first_row + min(r, n_rows - 1));
    const bool on = r < n_rows && x.on;
    const bool any = __builtin_amdgcn_ballot_w64(on) != 0;
    const int32_t grp = chunk / C.group_blocks;
    uint32_t row = 0, fe = 0;
    if (any) {
        row = rank_row(D, grp, x.kv, x.bs);
        fe = rank_lane(D, grp, x.xf, x.xe);
    }
    asm volatile("" ::"v"(row), "v"(fe));
    float* to = values + r / kWave * D.n_trees * kWave + lane_id();
    int cur = 0;
    for (int32_t t = t0; t < t1; t += tb, cur ^= 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t + tb < t1) stage_trees<true>(D, t + tb, min(tb, t1 - t - tb), lds_addr(smem) + (cur ^ 1) * buf_bytes, wave, WAVES);
        if (!any) continue;
        const int32_t cnt = min(tb, t1 - t);
        const uint32_t tree = lds_addr(smem) + cur * buf_bytes;
        float* o = to + (int64_t)t * kWave;
        int32_t q = 0;
        for (; q + 4 <= cnt; q += 4) put_leaves<4>(tree + q * bytes, bytes, D.depth, row, fe, o + q * kWave, on);
        for (; q + 2 <= cnt; q += 2) put_leaves<2>(tree + q * bytes, bytes, D.depth, row, fe, o + q * kWave, on);
        if (q < cnt) put_leaves<1>(tree + q * bytes, bytes, D.depth, row, fe, o + q * kWave, on);
    }
}

constexpr int kSumWaves = 8;
constexpr int kSumTrees = 32;                      // values in flight a lane
constexpr int kSumSeg = kSumWaves * kSumTrees;     // trees per LDS buffer

template <RowKind KIND>
__global__ __launch_bounds__(kSumWaves* kWave) void forest_sum_kernel(const float* __restrict__ values, int32_t n_trees, float base, SmallParams P,
                                                                      int64_t first_row, int64_t n_rows) {
    extern __shared__ float seg[];                 // [2][kSumSeg][64]
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int64_t r = (int64_t)blockIdx.x * kWave + lane;
    const float* from = values + (int64_t)blockIdx.x * n_trees * kWave + lane;
    float acc = base;
    int cur = 0;
    for (int32_t t0 = 0; t0 < n_trees; t0 += kSumSeg, cur ^= 1) {
        float* buf = seg + cur * kSumSeg * kWave;
        const int32_t cnt = min(kSumSeg, n_trees - t0);
        // wavefront w takes trees w, w + 8, ... of the segment
        float v[kSumTrees];
#pragma unroll
        for (int i = 0; i < kSumTrees; ++i) {
            const int32_t t = i * kSumWaves + wave;
            if (t < cnt) v[i] = from[(int64_t)(t0 + t) * kWave];
        }
#pragma unroll
        for (int i = 0; i < kSumTrees; ++i) {
            const int32_t t = i * kSumWaves + wave;
            if (t < cnt) buf[t * kWave + lane] = v[i];
        }
        // one barrier a segment: wavefront 0 adds this buffer while the
        // others fetch into the other one, and reaches the next barrier
        // before this buffer is written again
        __syncthreads();
        if (wave == 0) {
            int32_t t = 0;
            for (; t + 16 <= cnt; t += 16) {
                float u[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] = buf[(t + i) * kWave + lane];
#pragma unroll
                for (int i = 0; i < 16; ++i) acc += u[i];
            }
            for (; t < cnt; ++t) acc += buf[t * kWave + lane];
        }
    }
    if (wave != 0 || r >= n_rows) return;
    const int64_t i = first_row + r;
    if (KIND == kColumnRows && P.fidx && P.fidx[i / P.H] < 0) return;
    P.out[i] = acc;
}

// Bytes of scratch a slice takes at most.
constexpr size_t kSmallScratchBytes = (size_t)64 << 20;
constexpr int64_t kSliceRows = 1024;               // a slice is whole tiles

// More than 64 KiB of dynamic LDS has to be asked for (a call into the runtime
// that these short calls otherwise save).
hipError_t allow_lds(const void* kern, size_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

int64_t slice_rows(int32_t n_trees, int64_t n_rows) {
    const int64_t most = (int64_t)(kSmallScratchBytes / sizeof(float)) / std::max(1, n_trees) / kSliceRows * kSliceRows;
    const int64_t all = (n_rows + kSliceRows - 1) / kSliceRows * kSliceRows;
    return std::min(most, all);
}

template <RowKind KIND, int WAVES>
hipError_t launch_leaves(const ForestDev& f, const SmallParams& p, int64_t first, int64_t n, float* values,
                         hipStream_t stream) {
    const int64_t tiles = (n + WAVES * kWave - 1) / (WAVES * kWave);
    // enough chunks of trees for about kWorkgroups workgroups, at least 8 trees each
    constexpr int64_t kWorkgroups = 1024 * 4 / WAVES;
    const int64_t want = std::max<int64_t>(1, kWorkgroups / tiles);
    const int32_t chunk = (int32_t)std::max<int64_t>(8, (f.n_trees + want - 1) / want);
    const TreeBlocks C = tree_blocks(f.n_trees, f.group_trees, std::min(chunk, f.group_trees));
    const uint32_t bytes = staged_bytes<true>(f.depth);
    // two buffers in a share of the CU's LDS that leaves it full of wavefronts
    const size_t budget = std::max((size_t)80 * 1024 * WAVES / 16, std::min<size_t>(8 * (size_t)bytes, 64 * 1024));
    int32_t tb = C.tb;
    while (tb > 1 && 2 * (size_t)stage_buffer_bytes(tb, bytes) > budget) tb -= tb > 4 ? (tb + 3) % 4 + 1 : 1;
    const size_t lds = (C.tb > tb ? 2 : 1) * (size_t)stage_buffer_bytes(tb, bytes);
    const auto kern = forest_leaves_kernel<KIND, WAVES>;
    const hipError_t e = allow_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)C.n_blocks), dim3(WAVES * kWave), lds, stream,
                       rank_dev(f), C, tb, p, first, n, values);
    return hipGetLastError();
}

template <RowKind KIND>
hipError_t launch_small(const ForestDev& f, const SmallParams& p, int64_t n_rows, void* ws, hipStream_t stream) {
    float* values = (float*)ws;
    const int64_t step = slice_rows(f.n_trees, n_rows);
    const size_t lds = (f.n_trees > kSumSeg ? 2 : 1) * (size_t)std::min(f.n_trees, kSumSeg) * kWave * sizeof(float);
    const auto sum = forest_sum_kernel<KIND>;
    hipError_t e = allow_lds((const void*)sum, lds);
    for (int64_t first = 0; first < n_rows && e == hipSuccess; first += step) {
        const int64_t n = std::min(step, n_rows - first);
        // a large tile shares a staged chunk among more rows; a small one
        // spreads few rows over more CUs
        e = n * f.n_trees >= (int64_t)1 << 22 ? launch_leaves<KIND, 16>(f, p, first, n, values, stream)
                                              : launch_leaves<KIND, 4>(f, p, first, n, values, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(sum, dim3((unsigned)((n + kWave - 1) / kWave)), dim3(kSumWaves * kWave), lds, stream, values,
                           f.n_trees, f.base_score, p, first, n);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

size_t small_bytes(const ForestDev& f, const SmallParams& p) {
    if (!f.records || f.n_trees == 0) return 0;
    const int64_t n = small_rows(p);
    if (n <= 0 || slice_rows(f.n_trees, n) == 0) return 0;
    // Up to this many rows the two launches take less time than one that
    // leaves CUs idle.  Per row and tree they cost about 3.3 ps (depth 6 to
    // 8; 4 at 10); the others, however few the rows, a chain of walks per tree:
    // 0.4 us at depth 8 for the column kernel, 0.84 us (1.4 at depth 10) for
    // the grid kernel at 8 rows a wavefront.  (500 trees of depth 8: 100 000
    // rows 178 against 203 us, 300 000 rows 483 against 403; the grid of 4 boards
    // x 64 x 1024 436 against 421, 16 boards 1559 against 546.)
    if (n > (p.grid ? 30000 : 15000) * (int64_t)f.depth) return 0;
    // ... and from this many levels on (three more a tree; twice as many from
    // depth 10, where a buffer holds few trees): the second launch takes about
    // 5 us, which few trees' walks are over in.  (us, two launches / one: the
    // grid of one board x 17 x 512 with 20 trees of depth 4 11 / 11, 40 11 / 17, 8
    // boards with 20 of 8 18 / 16, 40 24 / 27; 1024 rows with 20 of 8 12 / 11, 40 12 /
    // 19; a search on one board x 16 with 30 of 8 70 / 59, 40 69 / 73; on 8 x 512
    // with 20 of 8 78 / 75, 30 87 / 100, 10 of 10 90 / 80, 15 92 / 96.)
    const int64_t levels = (int64_t)f.n_trees * (f.depth < 10 ? f.depth + 3 : 2 * f.depth);
    // (No more than that on larger calls, where the grid kernel's time depends on
    // how KV and batch move: 60 trees of depth 5, one board x 64 x 2048 with
    // KV drawn anew at every iteration 34 / 133.)
    const int64_t most = p.grid ? std::min<int64_t>(150 + n / 300, 270)
                       : n < 1024 ? 400 : std::min<int64_t>(250 + n / 300, 350);
    if (levels <= most) return 0;
    return (size_t)slice_rows(f.n_trees, n) * f.n_trees * sizeof(float);
}

hipError_t launch_forest_small(const ForestDev& f, const SmallParams& p, void* ws, hipStream_t stream) {
    const int64_t n = small_rows(p);
    return p.rows ? launch_small<kOwnRows>(f, p, n, ws, stream)
           : p.grid ? launch_small<kGridRows>(f, p, n, ws, stream)
                    : launch_small<kColumnRows>(f, p, n, ws, stream);
}

}  // namespace tl
