// Stage 2: the performance model M (Sec. 4.3.1), a gradient-boosted tree
// ensemble, evaluated on fp32 feature rows.  Every kernel here computes, for
// each row, base + the leaf of every tree as an fp32 running sum in tree
// order (every add rounded to nearest even).
//
// Grid kernels evaluate the rows of the projection grid without
// materializing them: row (s, f, j) = (freq[f], kv[s][j], batch[s][j]
// [, engine[s]]).  One wavefront takes one scenario and J consecutive future
// iterations; its lanes are the candidate frequencies, so every lane sees the
// same (KV, batch) sequence.  For each tree (in order) a lane keeps the leaf
// reached by its previous row together with the KV / batch box of that leaf
// (the bounds its root-to-leaf path puts on those two features); the next row
// reuses the leaf while its (KV, batch) stays inside the box.  This is exact:
// frequency and engine size are fixed for the lane, so a row inside the box
// takes every decision of the path the same way.  Between consecutive future
// iterations KV and batch move little, so most rows cost a box test and one
// fp32 add per tree; a walk happens on roughly one row in twenty.
//
//   forest_grid_lds_kernel     (depth <= 11) A 1024-thread workgroup (16
//       wavefronts of 32, 16 or 8 iterations x 64 frequencies, see grid_rows)
//       walks the ensemble in blocks of trees staged in LDS buffers.  A tree is one rank record (nodes, leaf values,
//       leaf boxes; record_format.h), so a block is one contiguous copy, made
//       straight from global memory into LDS and handed from wavefront to
//       wavefront without block barriers (stage_acquire / stage_release).
//       Tree walks read LDS only, four vector instructions a level.
//       Trees are taken in pairs that share one box test (a row that leaves
//       it walks only the tree whose own box it left), and rows in groups of
//       eight whose (KV, batch) hull is tested before any single row.  Rows,
//       hulls and boxes are pairs of 16-bit ranks in one register: a row's
//       box test is a packed min, a packed max and a compare.  The
//       (scenario, chunk) items are ordered by an estimate of their walks,
//       so a workgroup's wavefronts do similar work.
//   forest_grid_global_kernel  (deeper trees) The same per-lane scheme with
//       nodes, leaves and boxes read from global memory, one row at a time.
//
// Device layout (built by tl_forest_create): nodes [T][2^d] (8 bytes:
// threshold bits, feature; the last entry of each tree is padding), leaves
// [T][2^d] fp32, and for 3-4 features the leaf boxes [T][2^d] (kv_lo, kv_hi,
// batch_lo, batch_hi) or, up to depth 11, the rank records of the LDS
// kernel.
//
// forest_rows_kernel evaluates arbitrary rows: each thread walks RPT
// consecutive rows through every tree (forests without LDS records; the
// others take the column kernel's staged walks).
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <mutex>

#include "device_util.h"
#include "tl_internal.h"
#include "forest_walk.h"

namespace tl {
namespace {

template <int NF>
__device__ __forceinline__ float pick(const float (&x)[4], uint32_t f) {
    if (NF == 1) return x[0];
    if (NF == 2) return f == 0 ? x[0] : x[1];
    if (NF == 3) return f == 0 ? x[0] : (f == 1 ? x[1] : x[2]);
    return f == 0 ? x[0] : (f == 1 ? x[1] : (f == 2 ? x[2] : x[3]));
}

// grid row features: 0 frequency, 1 KV, 2 batch, 3 engine size
template <int NF>
__device__ __forceinline__ float pick_grid(uint32_t ft, float xf, float kv, float bs, float xe) {
    if (NF == 3) return ft == 0 ? xf : (ft == 1 ? kv : bs);
    return ft == 0 ? xf : (ft == 1 ? kv : (ft == 2 ? bs : xe));
}

template <int NF, int RPT>
__global__ __launch_bounds__(256) void forest_rows_kernel(const uint2* __restrict__ nodes,
                                                          const float* __restrict__ leaves,
                                                          int32_t n_trees, int32_t depth, float base,
                                                          const float* __restrict__ rows, int64_t n_rows,
                                                          float* __restrict__ out) {
    const int64_t r0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * RPT;
    if (r0 >= n_rows) return;
    const int nr = (int)min((int64_t)RPT, n_rows - r0);
    float x[RPT][4];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[r][c] = 0.0f;
        if (r < nr) {
#pragma unroll
            for (int c = 0; c < NF; ++c) x[r][c] = rows[(r0 + r) * NF + c];
        }
    }
    float acc[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) acc[r] = base;
    const int32_t n_int = (1 << depth) - 1;
    const int32_t n_leaf = 1 << depth;
    for (int32_t t = 0; t < n_trees; ++t) {
        const uint2* nt = nodes + (int64_t)t * n_leaf;
        const float* lt = leaves + (int64_t)t * n_leaf;
        int32_t k[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) k[r] = 0;
        for (int32_t level = 0; level < depth; ++level) {
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const uint2 nd = nt[k[r]];
                const float v = pick<NF>(x[r], nd.y);
                k[r] = 2 * k[r] + ((v < __uint_as_float(nd.x)) ? 1 : 2);
            }
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) acc[r] += lt[k[r] - n_int];
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r)
        if (r < nr) out[r0 + r] = acc[r];
}

constexpr int kLdsJ = 32;                // future iterations per wavefront (LDS kernel)
constexpr int kLdsWaves = 16;            // wavefronts per workgroup
constexpr int kLdsThreads = kLdsWaves * kWave;
// Two workgroups share a CU: half its LDS each, and 64 registers a lane.
// Measured (ms a step; 1024 boards x 2048 iterations x 64 frequencies with
// 500 trees of depth 8 / 4096 x 1024 x 64 with 2000 of depth 10 / 256 x 4096 x
// 32 with 300 of depth 8): J = 32 at 8 wavefronts per SIMD 6.9 / 86.5 / 2.10;
// J = 40 at 6 7.5 / 86.8 / 2.26; J = 64 at 4 (one workgroup, the whole LDS)
// 8.7 / 84.4 / 2.42.  A longer chunk saves walks of first rows, more
// wavefronts hide the walks' chains of LDS reads; at 8 the VALU issues nearly
// all the time.
constexpr int kLdsWavesPerSimd = 8;
constexpr size_t kLdsBudget = 80 * 1024;
constexpr int kLdsBuffers = 2;           // tree buffers
constexpr int kOrderJ = 64;              // future iterations per entry of the work order
constexpr int kGlobalJ = 32;             // future iterations per wavefront (global kernel)

// Which (scenario, frequency group, iteration chunk) a wavefront evaluates.
struct GridItem {
    bool valid;
    int64_t s;
    int32_t f, j0, nj;
};

// Items are numbered scenario-fastest within an iteration chunk of J * PER
// rows, the PER items of one chunk next to each other: the wavefronts of one
// workgroup take the same chunk (and frequency group) of consecutive
// scenarios.
// How many walks a chunk needs follows how fast KV and batch change there;
// workgroups whose wavefronts do similar work lose less time waiting for
// their slowest wavefront to release a tree buffer.  With a work order
// (P.order), entry i of a frequency group takes
// the (scenario, chunk) pair order[i] instead: pairs sorted by estimated
// cost, most expensive first.
template <int J, int PER>
__device__ __forceinline__ GridItem grid_item(const GridParams& P, int64_t item) {
    const int32_t n_chunks = (P.H + J * PER - 1) / (J * PER);
    const int32_t n_fg = (P.F + kWave - 1) / kWave;   // (1 where a wavefront takes two parts of a chunk)
    GridItem g;
    g.valid = item < P.S * n_fg * n_chunks * PER;
    const int64_t it = g.valid ? item / PER : 0;
    const int32_t part = g.valid ? (int32_t)(item % PER) : 0;
    const int64_t n_pairs = P.S * n_chunks;
    int32_t chunk;
    if (P.order) {
        const uint32_t code = P.order[it % n_pairs];
        g.s = code / (uint32_t)n_chunks;
        chunk = (int32_t)(code % (uint32_t)n_chunks);
        g.f = (int32_t)(it / n_pairs) * kWave + lane_id();
    } else {
        g.s = it % P.S;
        const int64_t rest = it / P.S;
        g.f = (int32_t)(rest % n_fg) * kWave + lane_id();
        chunk = (int32_t)(rest / n_fg);
    }
    g.j0 = (chunk * PER + part) * J;
    if (g.j0 >= P.H) {   // the last chunk may hold fewer items
        g.valid = false;
        g.j0 = 0;
    }
    g.nj = min(J, P.H - g.j0);
    return g;
}

// ---------------------------------------------------------------- LDS-staged

// A wavefront-uniform value read into a scalar register: the compiler's lane
// read, with the empty asm statements hiding how x was computed and pinning
// the result to the scalar register file (the compiler would otherwise
// rematerialize it in vector registers).
__device__ __forceinline__ uint32_t to_sgpr(uint32_t x) {
    asm volatile("" : "+v"(x));
    uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)x);
    asm volatile("" : "+s"(r));
    return r;
}

constexpr int kRowGroup = 8;   // rows whose (KV, batch) hull is tested as one

// Adds the leaves of NT (1 or 2) consecutive staged trees (rec_bytes apart,
// the first at LDS byte address `tree`) to the J row sums of a wavefront, in
// tree order.  hull[g] is the box of the rows of group g; rows4 holds the
// rows' rank pairs, four per 16 bytes.  A lane keeps the values of the leaves
// its walks reached, their boxes and the intersection of the boxes.  A group
// whose hull lies inside that intersection on every lane needs only its adds;
// other groups test row by row.  A lane whose row leaves the intersection
// walks only the trees whose own box it left (both in one pass when the
// wavefront needs both) and reads the new leaves' values and boxes.
template <int J, int NT, class Hulls>
__device__ __forceinline__ void eval_trees(uint32_t tree, uint32_t rec_bytes, int32_t depth, const uint4* rows4,
                                           Hulls&& hulls, uint32_t fe, const uint32_t (&first)[NT], float (&acc)[J]) {
    static_assert(J % kRowGroup == 0 && kRowGroup % 4 == 0, "whole row groups");
    static_assert(NT == 1 || NT == 2, "one tree or a pair");
    // the rows are re-read from LDS for each group that needs them rather
    // than held in registers across the tree loop
    asm volatile("" ::: "memory");
    const uint32_t tree1 = tree + rec_bytes;
    // a pair's own leaf boxes beside their intersection: after a walk only
    // the walked tree's box is read again
    Box box, b0, b1 = empty_box();
    float v[NT];
    v[0] = leaf_value(first[0]);
    b0 = leaf_box(first[0], tree);
    box = b0;
    if (NT == 2) {
        v[NT - 1] = leaf_value(first[NT - 1]);
        b1 = leaf_box(first[NT - 1], tree1);
        box = box_meet(b0, b1);
    }
#pragma unroll
    for (int gi = 0; gi < J / kRowGroup; ++gi) {
        const Box hull = hulls(gi);
        const uint32_t outside = pair_above(hull.lo, box.lo) | pair_above(box.hi, hull.hi);
        const bool test_rows = __builtin_amdgcn_ballot_w64(outside != 0) != 0;   // wavefront-uniform
        uint4 q = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < kRowGroup; ++i) {
            if (test_rows) {
                if ((i & 3) == 0) {
                    // four rows per read; the barrier keeps the compiler from
                    // hoisting all reads of the group (registers)
                    asm volatile("" ::: "memory");
                    q = rows4[gi * (kRowGroup / 4) + i / 4];
                }
                const uint32_t row = (i & 3) == 0 ? q.x : (i & 3) == 1 ? q.y : (i & 3) == 2 ? q.z : q.w;
                if (!in_box(box, row)) {
                    if (NT == 1) {
                        uint32_t k[1];
                        walk<1>(tree, rec_bytes, depth, row, fe, k);
                        v[0] = leaf_value(k[0]);
                        box = leaf_box(k[0], tree);
                    } else {
                        const bool n0 = !in_box(b0, row);
                        const bool n1 = !in_box(b1, row);
                        if (__builtin_amdgcn_ballot_w64(n0) != 0 && __builtin_amdgcn_ballot_w64(n1) != 0) {
                            uint32_t k[2];
                            walk<2>(tree, rec_bytes, depth, row, fe, k);
                            if (n0) {
                                v[0] = leaf_value(k[0]);
                                b0 = leaf_box(k[0], tree);
                            }
                            if (n1) {
                                v[NT - 1] = leaf_value(k[1]);
                                b1 = leaf_box(k[1], tree1);
                            }
                        } else {
                            if (n0) {
                                uint32_t k[1];
                                walk<1>(tree, rec_bytes, depth, row, fe, k);
                                v[0] = leaf_value(k[0]);
                                b0 = leaf_box(k[0], tree);
                            }
                            if (n1) {
                                uint32_t k[1];
                                walk<1>(tree1, rec_bytes, depth, row, fe, k);
                                v[NT - 1] = leaf_value(k[0]);
                                b1 = leaf_box(k[0], tree1);
                            }
                        }
                        box = box_meet(b0, b1);
                    }
                }
            }
            float& a = acc[gi * kRowGroup + i];
#pragma unroll
            for (int t = 0; t < NT; ++t) a += v[t];
            // consume the sum here so the adds are not sunk past later walks
            // (that would keep leaf values live)
            asm volatile("" ::"v"(a));
        }
    }
}

// PARTS: a wavefront takes PARTS (1 or 2) consecutive parts of J rows of one
// scenario, 64 / PARTS lanes each: with at most 32 frequencies two parts fill
// its lanes.  A row, and a group's hull, then differ between the halves: the
// hulls are read from LDS instead of held in scalar registers.
template <int J, int PARTS>
__global__ __launch_bounds__(kLdsThreads, kLdsWavesPerSimd) void forest_grid_lds_kernel(RankDev D, TreeBlocks B,
                                                                                             GridParams P) {
    constexpr int kRows = J * PARTS, kLanes = kWave / PARTS, kGroups = J / kRowGroup;
    static_assert(kRows <= kWave, "one lane ranks each row");
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t rec_bytes = rank_record_bytes(D.depth);
    const uint32_t buf_bytes = stage_buffer_bytes(B.tb, rec_bytes);

    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int64_t item = __builtin_amdgcn_readfirstlane((int64_t)blockIdx.x * kLdsWaves + wave);
    GridItem g = grid_item<kRows, kOrderJ / kRows>(P, item);
    const int32_t F = P.F, H = P.H;
    const int part = lane / kLanes;
    if (PARTS > 1) g.f = lane % kLanes;
    const int32_t j0 = g.j0 + part * J, nj = min(J, H - j0);   // the lane's rows (nj <= 0: none)
    const bool active = g.valid && g.f < F && nj > 0;
    // the rank pairs of this wavefront's rows are the same for every lane of a
    // part; they sit in LDS after the tree buffers and are read as broadcasts,
    // after them the groups' hulls (PARTS > 1)
    constexpr int kWords = kRows + (PARTS > 1 ? 2 * kGroups * PARTS : 0);
    uint32_t* rows = (uint32_t*)(smem + kLdsBuffers * buf_bytes) + wave * kWords;
    StageSync* sync = (StageSync*)(smem + kLdsBuffers * buf_bytes + (size_t)kLdsWaves * kWords * sizeof(uint32_t));
    if (threadIdx.x == 0) stage_sync_init<kLdsBuffers>(sync);

    // staging: block 0 by every wavefront before the barrier, the others
    // handed over without barriers (stage_acquire / stage_release)
    float acc[J];
#pragma unroll
    for (int jj = 0; jj < J; ++jj) acc[jj] = D.base;
    if (B.n_blocks > 0) stage_block(D, B, 0, lds_addr(smem), wave, kLdsWaves);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    bool sync_ok = true;
    for (int32_t grp = 0; grp < D.n_groups; ++grp) {
        // this group's ranks of the lane's frequency and engine size (a NaN
        // ranks above every threshold: every right turn, as in a plain walk)
        // and of row `lane` (rows past the horizon repeat its last)
        const int32_t j = min(g.j0 + min(lane, kRows - 1), H - 1);
        const uint32_t fe = rank_lane(D, grp, P.freqs[g.f < F ? g.f : F - 1], P.engine ? P.engine[g.s] : 0.0f);
        const uint32_t own = rank_row(D, grp, (float)P.kv[g.s * H + j], (float)P.batch[g.s * H + j]);
        if (lane < kRows) rows[lane] = own;
        asm volatile("" ::: "memory");
        // per row group, the box of its rows
        const uint4* rows4 = (const uint4*)(rows + part * J);
        auto group_hull = [&](int gi) {
            uint32_t lo = 0xffffffffu, hi = 0;
#pragma unroll
            for (int i = 0; i < kRowGroup / 4; ++i) {
                const uint4 q = rows4[gi * (kRowGroup / 4) + i];
                lo = pair_min(lo, pair_min(pair_min(q.x, q.y), pair_min(q.z, q.w)));
                hi = pair_max(hi, pair_max(pair_max(q.x, q.y), pair_max(q.z, q.w)));
            }
            return Box{lo, hi};
        };
        Box hull[kGroups];
        const uint2* hull_at = (const uint2*)(rows + kRows) + part * kGroups;
#pragma unroll
        for (int gi = 0; gi < kGroups; ++gi) {
            const Box h = group_hull(gi);
            if (PARTS == 1) {   // wavefront-uniform
                hull[gi].lo = to_sgpr(h.lo);
                hull[gi].hi = to_sgpr(h.hi);
            } else if (lane % kLanes == 0) {
                ((uint2*)hull_at)[gi] = make_uint2(h.lo, h.hi);
            }
        }
        auto hulls = [&](int gi) {
            if (PARTS == 1) return hull[gi];
            asm volatile("" ::: "memory");   // read when needed, not held in registers
            const uint2 h = hull_at[gi];
            return Box{h.x, h.y};
        };
        // the ranks are complete before this wavefront stages again: the
        // walks then never wait for a copy in flight
        asm volatile("" ::"v"(fe) : "memory");
        const int32_t b_end = min((grp + 1) * B.group_blocks, B.n_blocks);
        for (int32_t b = grp * B.group_blocks; b < b_end; ++b) {
            const uint32_t buf = lds_addr(smem) + (uint32_t)(b % kLdsBuffers) * buf_bytes;
            if (b > 0) sync_ok &= stage_acquire<kLdsBuffers>(sync, b, kLdsWaves, D, B, buf);
            if (g.valid) {
                const int32_t cnt = block_count(D, B, b, block_first(D, B, b));
                // Trees are taken two at a time and a lane keeps the
                // intersection of the two leaf boxes: a row inside it reaches
                // both leaves again.  When a row leaves it, both trees are
                // walked in one pass, so the two chains of dependent LDS
                // reads overlap.
                int32_t tt = 0;
                const uint32_t row0 = rows4[0].x;
                auto pair = [&](uint32_t tree, const uint32_t(&first)[2]) {
                    eval_trees<J, 2>(tree, rec_bytes, D.depth, rows4, hulls, fe, first, acc);
                };
                // the first row's walks four trees at once (37 boards x 23 x
                // 777, 250 trees of depth 7: 218 -> 207 us a step; 256 x 32 x
                // 4096, 300 of depth 8: 1528 -> 1497)
                for (; tt + 3 < cnt; tt += 4) {
                    const uint32_t tree = buf + tt * rec_bytes;
                    uint32_t k[4];
                    walk<4>(tree, rec_bytes, D.depth, row0, fe, k);
                    pair(tree, {k[0], k[1]});
                    pair(tree + 2 * rec_bytes, {k[2], k[3]});
                }
                for (; tt + 1 < cnt; tt += 2) {
                    const uint32_t tree = buf + tt * rec_bytes;
                    uint32_t k[2];
                    walk<2>(tree, rec_bytes, D.depth, row0, fe, k);
                    pair(tree, k);
                }
                if (tt < cnt) {
                    const uint32_t tree = buf + tt * rec_bytes;
                    uint32_t k[1];
                    walk<1>(tree, rec_bytes, D.depth, row0, fe, k);
                    eval_trees<J, 1>(tree, rec_bytes, D.depth, rows4, hulls, fe, k, acc);
                }
            }
            stage_release<kLdsBuffers>(sync, b, kLdsWaves);
        }
    }
    if (active) {
        float* o = P.out + ((int64_t)g.s * F + g.f) * H + j0;
#pragma unroll
        for (int jj = 0; jj < J; ++jj)
            if (jj < nj) o[jj] = sync_ok ? acc[jj] : __builtin_nanf("");
    }
}

// ------------------------------------------------------------ global memory

constexpr int kGlobalWaves = 4;

template <int NF, int J>
__global__ __launch_bounds__(256) void forest_grid_global_kernel(const uint2* __restrict__ nodes,
                                                                 const float* __restrict__ leaves,
                                                                 const float4* __restrict__ boxes,
                                                                 int32_t n_trees, int32_t depth, float base,
                                                                 GridParams P) {
    __shared__ float2 kvb[kGlobalWaves][J];
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int64_t item = __builtin_amdgcn_readfirstlane((int64_t)blockIdx.x * kGlobalWaves + wave);
    const GridItem g = grid_item<J, 1>(P, item);
    const int32_t F = P.F, H = P.H;
    const bool active = g.valid && g.f < F;
    const float xf = P.freqs[g.f < F ? g.f : F - 1];
    const float xe = (NF == 4) ? P.engine[g.s] : 0.0f;
    if (lane < J) {
        const int32_t j = g.j0 + min(lane, g.nj - 1);
        kvb[wave][lane] = make_float2((float)P.kv[g.s * H + j], (float)P.batch[g.s * H + j]);
    }
    __syncthreads();
    if (!g.valid) return;

    float acc[J];
#pragma unroll
    for (int jj = 0; jj < J; ++jj) acc[jj] = base;
    const int32_t n_int = (1 << depth) - 1;
    const int32_t n_leaf = 1 << depth;
    for (int32_t t = 0; t < n_trees; ++t) {
        const uint2* nt = nodes + (int64_t)t * n_leaf;
        const float* lv = leaves + (int64_t)t * n_leaf;
        const float4* bx = boxes + (int64_t)t * n_leaf;
        float lo_k = INFINITY, hi_k = -INFINITY, lo_b = INFINITY, hi_b = -INFINITY;
        float val = 0.0f;
#pragma unroll
        for (int jj = 0; jj < J; ++jj) {
            const float2 v2 = kvb[wave][jj];
            const bool hit = (v2.x >= lo_k) & (v2.x < hi_k) & (v2.y >= lo_b) & (v2.y < hi_b);
            if (!hit) {
                int32_t k = 0;
                for (int32_t level = 0; level < depth; ++level) {
                    const uint2 nd = nt[k];
                    const float x = pick_grid<NF>(nd.y, xf, v2.x, v2.y, xe);
                    k = 2 * k + ((x < __uint_as_float(nd.x)) ? 1 : 2);
                }
                const int32_t leaf = k - n_int;
                val = lv[leaf];
                const float4 b = bx[leaf];
                lo_k = b.x;
                hi_k = b.y;
                lo_b = b.z;
                hi_b = b.w;
            }
            acc[jj] += val;
        }
    }
    if (active) {
        float* o = P.out + ((int64_t)g.s * F + g.f) * H + g.j0;
#pragma unroll
        for (int jj = 0; jj < J; ++jj)
            if (jj < g.nj) o[jj] = acc[jj];
    }
}

template <int NF>
hipError_t launch_nf(const ForestDev& f, const float* rows, int64_t n_rows, float* out, hipStream_t stream) {
    constexpr int RPT = 4;
    constexpr int TPB = 256;
    const int64_t threads = (n_rows + RPT - 1) / RPT;
    const int64_t blocks = (threads + TPB - 1) / TPB;
    if (!grid_fits(blocks, TPB)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((forest_rows_kernel<NF, RPT>), dim3((unsigned)blocks), dim3(TPB), 0, stream,
                       f.nodes, f.leaves, f.n_trees, f.depth, f.base_score, rows, n_rows, out);
    return hipGetLastError();
}

// Trees per staged block for the LDS kernel: the buffers and the wavefronts'
// rows must fit the LDS budget.  0 = the LDS kernel cannot run.
int32_t lds_trees_per_block(const ForestDev& f, size_t budget, size_t* lds_bytes) {
    if (!f.records || f.depth > kMaxRecordDepth) return 0;
    const uint32_t rec_bytes = rank_record_bytes(f.depth);
    // (two parts: 64 rows and 8 hulls a wavefront)
    const size_t head = (size_t)kLdsWaves * (kWave + 16) * sizeof(uint32_t) + sizeof(StageSync);
    auto fits = [&](int32_t tb) { return kLdsBuffers * (size_t)stage_buffer_bytes(tb, rec_bytes) + head <= budget; };
    // whole pairs of trees where two fit
    int32_t tb = 64;
    while (tb > 1 && !fits(tb)) tb -= tb > 2 ? 2 : 1;
    if (!fits(tb)) return 0;
    *lds_bytes = kLdsBuffers * (size_t)stage_buffer_bytes(tb, rec_bytes) + head;
    return tb;
}

// Parts of a chunk a wavefront takes: two where their frequencies fit.
int grid_parts(const GridParams& g) { return g.F <= kWave / 2 ? 2 : 1; }

int64_t grid_workgroups(const GridParams& g, int J) {
    const int64_t n_chunks = (g.H + kOrderJ - 1) / kOrderJ;
    const int64_t n_fg = (g.F + kWave - 1) / kWave;
    const int64_t items = g.S * n_fg * n_chunks * (kOrderJ / (J * grid_parts(g)));
    return (items + kLdsWaves - 1) / kLdsWaves;
}

template <int J, int PARTS>
hipError_t launch_grid_lds(const ForestDev& f, const GridParams& g, int32_t tb, size_t lds, hipStream_t stream) {
    const auto kern = forest_grid_lds_kernel<J, PARTS>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t blocks = grid_workgroups(g, J);
    if (!grid_fits(blocks, kLdsThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kLdsThreads), lds, stream, rank_dev(f),
                       tree_blocks(f.n_trees, f.group_trees, tb), g);
    return hipGetLastError();
}

// Rows per wavefront: 8 or 16 where 32 would leave CUs without their two
// workgroups.  Shorter chunks walk more first rows, whose share grows with the
// depth: 8 while its workgroups x depth stay within 16 per CU, then 16.
// Measured (us a step at 8 / 16 / 32 rows): 64 boards x 64 x 1024 with 500 trees
// of depth 8 (512 workgroups at 8 rows) 573 / 779 / 1054, with 2000 of depth 10
// 4133 / 3366 / 4563, 256 boards of the former 1999 / 1427 / 1265.
// *ordered: 32 rows, and more workgroups than start at once: only then does a
// work order pay.  *alone: at most one workgroup per CU.
void grid_rows(const ForestDev& f, const GridParams& g, int* J, bool* ordered, bool* alone) {
    const int64_t cus = f.cus;
    auto fits = [&](int rows) { return grid_workgroups(g, rows) * std::max(f.depth, 1) <= 16 * cus; };
    *J = fits(8) ? 8 : fits(16) ? 16 : kLdsJ;
    *ordered = *J == kLdsJ && grid_workgroups(g, kLdsJ) > 2 * cus;
    *alone = grid_workgroups(g, *J) <= cus;
}

template <int NF>
hipError_t launch_grid_global(const ForestDev& f, const GridParams& g, hipStream_t stream) {
    const int64_t n_chunks = (g.H + kGlobalJ - 1) / kGlobalJ;
    const int64_t n_fg = (g.F + kWave - 1) / kWave;
    const int64_t items = g.S * n_fg * n_chunks;
    const int64_t blocks = (items + kGlobalWaves - 1) / kGlobalWaves;
    if (!grid_fits(blocks, kGlobalWaves * kWave)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((forest_grid_global_kernel<NF, kGlobalJ>), dim3((unsigned)blocks), dim3(kGlobalWaves * kWave),
                       0, stream, f.nodes, f.leaves, f.kvb_box, f.n_trees, f.depth, f.base_score, g);
    return hipGetLastError();
}

}  // namespace


namespace {

// Estimated cost of each pair of a work order, (scenario, J consecutive
// iterations): by how many thresholds' ranks KV and batch move from one row
// to the next in the first rank group (each threshold crossed changes a
// decision of some tree, which may cost a walk).  One wavefront per pair, one
// row a lane.  Writes cost[i] and the pair's code i = s * n_chunks + chunk.
// (One thread per pair, searching quantiles of the thresholds for its rows in
// turn, took 130 us however few the pairs.)
constexpr int kCostWaves = 4;

__global__ __launch_bounds__(kCostWaves* kWave) void pair_cost_kernel(RankDev D, const int32_t* __restrict__ kv,
                                                                      const int32_t* __restrict__ batch, int64_t n,
                                                                      int32_t H, int32_t J,
                                                                      uint32_t* __restrict__ cost,
                                                                      uint32_t* __restrict__ code) {
    const int64_t pair = (int64_t)blockIdx.x * kCostWaves + threadIdx.x / kWave;
    if (pair >= n) return;
    const int32_t n_chunks = (H + J - 1) / J;
    const int64_t s = pair / n_chunks;
    const int32_t j0 = (int32_t)(pair % n_chunks) * J, j1 = min(j0 + J, H);
    int32_t sum = 0, before = -1;   // the last rank pair of the step before
    for (int32_t j = j0; j < j1; j += kWave) {
        const int64_t i = s * H + min(j + lane_id(), j1 - 1);
        const int32_t r = (int32_t)rank_row(D, 0, (float)kv[i], (float)batch[i]);
        if (j == j0) before = __builtin_amdgcn_readfirstlane(r);
        const int32_t p = wave_shift_up1(r, before);
        sum += abs((r & 0xffff) - (p & 0xffff)) + abs((int32_t)((uint32_t)r >> 16) - (int32_t)((uint32_t)p >> 16));
        before = __builtin_amdgcn_readlane(r, kWave - 1);
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) {
        cost[pair] = (uint32_t)sum;
        code[pair] = (uint32_t)pair;
    }
}

}  // namespace

hipError_t pair_order_plan(const ForestDev& f, int64_t n, int64_t min_pairs, PairOrderPlan* p) {
    *p = PairOrderPlan{0, 0, 0, 0};
    if (!f.orderable || n < min_pairs || !grid_fits((n + kCostWaves - 1) / kCostWaves, kCostWaves * kWave))
        return hipSuccess;
    size_t temp = 0;
    const hipError_t e = hipcub::DeviceRadixSort::SortPairsDescending(
        nullptr, temp, (const uint32_t*)nullptr, (uint32_t*)nullptr, (const uint32_t*)nullptr, (uint32_t*)nullptr,
        (int)n, 0, 32, (hipStream_t)0);
    if (e != hipSuccess) return e;
    p->n = n;
    p->arr = ((size_t)n * sizeof(uint32_t) + 255) & ~(size_t)255;
    p->temp = temp;
    p->bytes = 4 * p->arr + temp;
    return hipSuccess;
}

hipError_t pair_order(const ForestDev& f, const PairOrderPlan& p, const int32_t* kv, const int32_t* batch, int32_t H,
                      int32_t J, void* ws, const uint32_t** order, hipStream_t stream) {
    unsigned char* base = (unsigned char*)ws;
    uint32_t* cost = (uint32_t*)base;
    uint32_t* code = (uint32_t*)(base + p.arr);
    uint32_t* cost_sorted = (uint32_t*)(base + 2 * p.arr);
    uint32_t* sorted = (uint32_t*)(base + 3 * p.arr);
    hipLaunchKernelGGL(pair_cost_kernel, dim3((unsigned)((p.n + kCostWaves - 1) / kCostWaves)),
                       dim3(kCostWaves * kWave), 0, stream, rank_dev(f), kv, batch, p.n, H, J, cost, code);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    size_t temp = p.temp;
    e = hipcub::DeviceRadixSort::SortPairsDescending(base + 4 * p.arr, temp, cost, cost_sorted, code, sorted, (int)p.n,
                                                     0, 32, stream);
    if (e != hipSuccess) return e;
    *order = sorted;
    return hipSuccess;
}

// Work order for the LDS grid kernel: (scenario, chunk) pairs by estimated
// cost, most expensive first, so a workgroup's wavefronts do similar work
// and the longest ones start first.
namespace {

hipError_t plan_order(const ForestDev& f, const GridParams& g, PairOrderPlan* p) {
    *p = PairOrderPlan{0, 0, 0, 0};
    size_t lds = 0;
    if (lds_trees_per_block(f, kLdsBudget, &lds) <= 0) return hipSuccess;   // the global kernel takes no order
    int J = 0;
    bool ordered = false;
    bool alone = false;
    grid_rows(f, g, &J, &ordered, &alone);
    if (!ordered) return hipSuccess;
    return pair_order_plan(f, g.S * ((g.H + kOrderJ - 1) / kOrderJ), 1, p);
}

}  // namespace

hipError_t grid_order_bytes(const ForestDev& f, const GridParams& g, size_t* bytes) {
    PairOrderPlan p;
    const hipError_t e = plan_order(f, g, &p);
    *bytes = e == hipSuccess ? p.bytes : 0;
    return e;
}

hipError_t launch_forest_grid(const ForestDev& f, const GridParams& g_in, void* ws, size_t ws_bytes,
                              hipStream_t stream) {
    GridParams g = g_in;
    g.order = nullptr;
    // Grids of more wavefronts than one launch takes go in parts of whole
    // scenarios, each a grid of its own.  (By a workgroup offset in the kernel's
    // parameters every grid paid for it: 256 boards x 32 x 4096 1115 -> 1136 us.)
    const int64_t waves = (g.F + kWave - 1) / kWave * (((int64_t)g.H + kOrderJ - 1) / kOrderJ) * (kOrderJ / kLdsJ);
    const int64_t most = std::max<int64_t>(1, (kMaxLaunchWaves - kLdsWaves) / waves);
    if (g.S > kMaxParts * most) return hipErrorInvalidConfiguration;
    if (g.S > most) {
        for (int64_t s0 = 0; s0 < g_in.S; s0 += most) {
            g = g_in;
            g.S = std::min(most, g_in.S - s0);
            g.kv += s0 * g.H;
            g.batch += s0 * g.H;
            if (g.engine) g.engine += s0;
            g.out += s0 * g.F * g.H;
            const hipError_t e = launch_forest_grid(f, g, ws, ws_bytes, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    size_t lds = 0;
    int32_t tb = lds_trees_per_block(f, kLdsBudget, &lds);
    if (tb <= 0) return f.n_features == 4 ? launch_grid_global<4>(f, g, stream) : launch_grid_global<3>(f, g, stream);
    PairOrderPlan p;
    hipError_t e = plan_order(f, g, &p);
    if (e != hipSuccess) return e;
    // the order only speeds the kernel up: without room for it the items
    // keep their natural numbering
    if (p.n > 0 && ws && ws_bytes >= p.bytes) {
        e = pair_order(f, p, g.kv, g.batch, g.H, kOrderJ, ws, &g.order, stream);
        if (e != hipSuccess) return e;
    }
    int J = 0;
    bool ordered = false;
    bool alone = false;
    grid_rows(f, g, &J, &ordered, &alone);
    // a workgroup with a CU to itself stages twice as many trees at a time
    if (alone) tb = lds_trees_per_block(f, 2 * kLdsBudget, &lds);
    if (grid_parts(g) == 2)
        return J == 32   ? launch_grid_lds<32, 2>(f, g, tb, lds, stream)
               : J == 16 ? launch_grid_lds<16, 2>(f, g, tb, lds, stream)
                         : launch_grid_lds<8, 2>(f, g, tb, lds, stream);
    return J == 32   ? launch_grid_lds<32, 1>(f, g, tb, lds, stream)
           : J == 16 ? launch_grid_lds<16, 1>(f, g, tb, lds, stream)
                     : launch_grid_lds<8, 1>(f, g, tb, lds, stream);
}

// Workspace of the grid kernel's work order for callers that cannot
// allocate (tl_forest_predict_grid_noalloc): one fixed array per device,
// shared by every such call on that device.  In host code `scratch` only
// names the symbol; its device address comes from hipGetSymbolAddress, once
// per device, and is kept in noalloc_ptr.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex noalloc_mutex;
void* noalloc_ptr[kMaxDevices];
}  // namespace

hipError_t noalloc_scratch(void** ptr) {
    *ptr = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(noalloc_mutex);
    if (!noalloc_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        noalloc_ptr[dev] = p;
    }
    *ptr = noalloc_ptr[dev];
    return hipSuccess;
}

hipError_t launch_forest_rows(const ForestDev& f, const float* rows, int64_t n_rows, float* out,
                              hipStream_t stream) {
    // 3- and 4-feature forests with LDS records: the staged walks of the
    // column kernel; otherwise walks from global memory
    const hipError_t e = launch_forest_rows_lds(f, rows, n_rows, out, stream);
    if (e != hipErrorNotSupported) return e;
    switch (f.n_features) {
        case 1: return launch_nf<1>(f, rows, n_rows, out, stream);
        case 2: return launch_nf<2>(f, rows, n_rows, out, stream);
        case 3: return launch_nf<3>(f, rows, n_rows, out, stream);
        default: return launch_nf<4>(f, rows, n_rows, out, stream);
    }
}

}  // namespace tl
