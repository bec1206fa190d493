// Node walks over tree records staged in LDS and leaf-box tests, shared by
// the forest kernels.  Records, rows and boxes are in rank space (layout and
// definitions: record_format.h).
//
// A node step is one 4-byte LDS read, a byte permute that picks the tested
// feature's 16-bit rank out of the row's two words, a 16-bit compare, a
// select and a shift-add to the child's address.  Nodes holding the fp32
// threshold and two permute selectors took a 16-byte read and six vector
// instructions; per tree the record was 24 instead of 16 bytes per leaf.
#pragma once

#include "device_util.h"
#include "tl_internal.h"

namespace tl {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) const u32x2 lds_u32x2;
typedef __attribute__((address_space(3))) const uint32_t lds_u32;
typedef __attribute__((address_space(3))) const float lds_f32;

// LDS byte address of a location in the kernel's dynamic LDS.
__device__ __forceinline__ uint32_t lds_addr(const unsigned char* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

// Pairs of 16-bit ranks, KV in the low half and batch in the high half.
__device__ __forceinline__ uint32_t pair_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pair_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// How far b lies above a in each half, 0 where it does not.
__device__ __forceinline__ uint32_t pair_above(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, b), __builtin_bit_cast(u16x2, a)));
}

// A leaf box: the lowest and highest rank pair inside it.
struct Box {
    uint32_t lo, hi;
};
__device__ __forceinline__ Box empty_box() { return Box{kEmptyBoxLo, kEmptyBoxHi}; }

// Whether a rank pair lies in a box: clamping it into the box leaves it as it
// is.  (With hi applied first, an empty box clamps everything to (65535,
// 65535), which no row is.)
__device__ __forceinline__ bool in_box(const Box& b, uint32_t row) {
    return pair_max(pair_min(row, b.hi), b.lo) == row;
}

// The intersection of two boxes that hold a common row.
__device__ __forceinline__ Box box_meet(const Box& a, const Box& b) {
    return Box{pair_max(a.lo, b.lo), pair_min(a.hi, b.hi)};
}

// The forest as the record kernels read it.
struct RankDev {
    const uint4* records;
    const RankGroup* groups;
    const float* dict;
    const uint16_t* starts;
    int32_t n_trees, depth, group_trees, n_groups;
    float base;
};

__host__ inline RankDev rank_dev(const ForestDev& f) {
    return RankDev{f.records, f.groups, f.dict, f.starts, f.n_trees, f.depth, f.group_trees, f.n_groups, f.base_score};
}

// A row's two words in group g: the rank pair of (KV, batch), and of
// (frequency, engine size).
__device__ __forceinline__ uint32_t rank_pair(const RankDev& D, int32_t g, int lo, int hi, float x, float y) {
    const RankFeature a = D.groups[g].f[lo], b = D.groups[g].f[hi];
    return rank_of(a, D.dict, D.starts, x) | rank_of(b, D.dict, D.starts, y) << 16;
}
__device__ __forceinline__ uint32_t rank_row(const RankDev& D, int32_t g, float kv, float bs) {
    return rank_pair(D, g, 1, 2, kv, bs);
}
__device__ __forceinline__ uint32_t rank_lane(const RankDev& D, int32_t g, float xf, float xe) {
    return rank_pair(D, g, 0, 3, xf, xe);
}

// A leaf reached by a walk, as the LDS byte address of its value: the walk's
// final address tree + 4 (2^d + L).  Its box is at tree + 8 (2^d + L).
__device__ __forceinline__ float leaf_value(uint32_t a) { return *(lds_f32*)(uintptr_t)a; }
__device__ __forceinline__ Box leaf_box(uint32_t a, uint32_t tree) {
    const u32x2 w = *(lds_u32x2*)(uintptr_t)(2u * a - tree);
    return Box{w.x, w.y};
}

// Staging of tree blocks: a block is consecutive trees of one group, one
// contiguous range of 16-byte words in global memory and in LDS.  It is
// copied in pieces of 64 lanes x 16 bytes straight from global memory into
// LDS (global_load_lds_dwordx4, no registers), wavefront w of n taking
// pieces w, w + n, ... (n = 1: one wavefront copies it all).  Lanes past the
// block's last word copy its first word into the buffer's padding (buffers
// are whole pieces), so no lane writes outside its buffer.
constexpr uint32_t kStagePiece = kWave * 16;

__host__ __device__ inline uint32_t stage_buffer_bytes(int32_t tb, uint32_t rec_bytes) {
    return ((uint32_t)tb * rec_bytes + kStagePiece - 1) / kStagePiece * kStagePiece;
}

// The blocks of a forest, tb trees each: group_blocks per group, a group's
// last block and the last group possibly short.
struct TreeBlocks {
    int32_t tb, group_blocks, n_blocks;
};
__host__ __device__ inline TreeBlocks tree_blocks(int32_t n_trees, int32_t group_trees, int32_t tb) {
    const int32_t gb = group_trees > 0 ? (group_trees + tb - 1) / tb : 1;
    const int32_t n_groups = group_trees > 0 ? (n_trees + group_trees - 1) / group_trees : 0;
    const int32_t last = n_groups > 0 ? n_trees - (n_groups - 1) * group_trees : 0;
    return TreeBlocks{tb, gb, n_groups > 0 ? (n_groups - 1) * gb + (last + tb - 1) / tb : 0};
}
// First tree and number of trees of block b.
__device__ __forceinline__ int32_t block_first(const RankDev& D, const TreeBlocks& B, int32_t b) {
    return b / B.group_blocks * D.group_trees + b % B.group_blocks * B.tb;
}
__device__ __forceinline__ int32_t block_count(const RankDev& D, const TreeBlocks& B, int32_t b, int32_t first) {
    return min(B.tb, min((b / B.group_blocks + 1) * D.group_trees, D.n_trees) - first);
}

// One piece: lane l copies the 16 bytes at its `src` to LDS byte address
// lds + 16 l (lds the same in every lane).  Issued as an instruction the
// compiler does not track, so it does not make the evaluation's LDS reads
// wait for the copy (they read other buffers); a kernel waits for its copies
// (vmcnt) before it hands the buffer over (a workgroup barrier, or
// publishing `ready` in stage_acquire), and has no other vector-memory load
// in flight inside its block loop.
__device__ __forceinline__ void stage_piece(const uint4* src, uint32_t lds) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds);   // wavefront-uniform by construction
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(base), "v"(src) : "memory", "m0");
}

// Bytes of a staged tree: the whole record, or (HALF) its nodes and leaf
// values only, for walks that never look at a box.
template <bool HALF>
__host__ __device__ inline uint32_t staged_bytes(int32_t depth) {
    const uint32_t whole = rank_record_bytes(depth);
    return HALF && depth > 0 ? whole / 2 : whole;
}

// Enqueues this wavefront's pieces of trees [first, first + cnt) into the LDS
// buffer at byte address dst.
template <bool HALF>
__device__ __forceinline__ void stage_trees(const RankDev& D, int32_t first, int32_t cnt, uint32_t dst, int wave,
                                            int n_waves) {
    const uint32_t rec_words = rank_record_bytes(D.depth) / 16u;
    const int32_t log_words = 31 - __builtin_clz(staged_bytes<HALF>(D.depth) / 16u);
    const uint32_t words = (uint32_t)cnt << log_words;
    const uint4* src = D.records + (int64_t)first * rec_words;
    const uint32_t n_pieces = (words + kWave - 1) / kWave;
    for (uint32_t pc = (uint32_t)wave; pc < n_pieces; pc += (uint32_t)n_waves) {
        const uint32_t i = pc * kWave + lane_id();
        const uint32_t w = i < words ? i : 0u;
        const uint32_t at = HALF ? (w >> log_words) * rec_words + (w & ((1u << log_words) - 1u)) : w;
        stage_piece(src + at, dst + pc * kStagePiece);
    }
}

// The same for block b.
template <bool HALF = false>
__device__ __forceinline__ void stage_block(const RankDev& D, const TreeBlocks& B, int32_t b, uint32_t dst, int wave,
                                            int n_waves) {
    const int32_t first = block_first(D, B, b);
    stage_trees<HALF>(D, first, block_count(D, B, b, first), dst, wave, n_waves);
}

// Hand-over of NB LDS buffers of tree blocks between the wavefronts of a
// workgroup without block barriers.  Block b lives in buffer b % NB; block 0
// is copied by every wavefront before the workgroup's one barrier.  Per
// buffer: `claimed` = the last block a wavefront took on to copy into it,
// `ready` = the last block whose copy is complete, `done` = how many
// (wavefront, block) pairs have finished with it.  The first wavefront that
// needs block b and finds it unclaimed claims it, waits until every
// wavefront has finished block b - NB (the buffer's previous occupant),
// copies the whole block, waits for its copy and publishes `ready`; the others
// wait for `ready`.  A wavefront can thus run up to NB - 1 blocks ahead of the
// slowest one instead of meeting it at every block.  Issue priority follows
// the order in which wavefronts finish a block: the later a wavefront leaves
// block b among its workgroup's, the higher its priority (s_setprio) while it
// evaluates block b + 1, and a wavefront that arrives at a block before its
// copy is there drops to the lowest; the oldest wavefronts of a SIMD would
// otherwise keep winning issue and the youngest set the pace.  Every wait is
// bounded (kSyncSpins sleeps); one that runs out makes stage_acquire return
// false, and the caller marks its results invalid, so every wavefront ends.
constexpr int kMaxStageBuffers = 4;
struct StageSync {
    int32_t claimed[kMaxStageBuffers];
    int32_t ready[kMaxStageBuffers];
    int32_t done[kMaxStageBuffers];
};
constexpr int32_t kSyncSpins = 1 << 20;

template <int NB = 2>
__device__ __forceinline__ void stage_sync_init(StageSync* sync) {
    sync->claimed[0] = 0;   // block 0: copied by every wavefront
    sync->ready[0] = 0;
    sync->done[0] = 0;
    for (int i = 1; i < NB; ++i) {
        sync->claimed[i] = i - NB;   // block i claims buffer i from "block i - NB"
        sync->ready[i] = -1;
        sync->done[i] = 0;
    }
}

__device__ __forceinline__ int32_t sync_load(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Makes block b >= 1 available in its buffer at LDS byte address buf;
// n_waves wavefronts share the buffers.
template <int NB = 2, bool HALF = false>
__device__ __forceinline__ bool stage_acquire(StageSync* sync, int32_t b, int n_waves, const RankDev& D,
                                              const TreeBlocks& B, uint32_t buf) {
    const int cur = b % NB;
    const int32_t need_done = n_waves * (b / NB);
    int32_t spins = 0;
    if (sync_load(&sync->ready[cur]) != b) __builtin_amdgcn_s_setprio(0);   // ahead of the others
    while (sync_load(&sync->ready[cur]) != b && spins < kSyncSpins) {
        int32_t won = 0;
        if (sync_load(&sync->claimed[cur]) == b - NB) {
            if (lane_id() == 0) {
                int32_t expect = b - NB;
                won = __hip_atomic_compare_exchange_strong(&sync->claimed[cur], &expect, b, __ATOMIC_ACQ_REL,
                                                           __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            won = __builtin_amdgcn_readfirstlane(won);
        }
        if (won) {
            while (sync_load(&sync->done[cur]) < need_done && spins < kSyncSpins) {
                __builtin_amdgcn_s_sleep(1);
                ++spins;
            }
            stage_block<HALF>(D, B, b, buf, 0, 1);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane_id() == 0) __hip_atomic_store(&sync->ready[cur], b, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
        ++spins;
    }
    return spins < kSyncSpins;
}

// This wavefront has finished with block b (its reads have all returned);
// n_waves share the buffers.
template <int NB = 2>
__device__ __forceinline__ void stage_release(StageSync* sync, int32_t b, int n_waves) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    int32_t before = 0;
    if (lane_id() == 0)
        before = __hip_atomic_fetch_add(&sync->done[b % NB], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    // how many wavefronts left block b before this one, in quarters
    const int32_t quarter = 4 * (__builtin_amdgcn_readfirstlane(before) % n_waves) / n_waves;
    if (quarter == 3) __builtin_amdgcn_s_setprio(3);
    else if (quarter == 2) __builtin_amdgcn_s_setprio(2);
    else if (quarter == 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// The leaves (lf[r][t], see leaf_value) that NR rows reach in NT consecutive
// staged trees (rec_bytes apart, the first at LDS byte address `tree`), all
// NR x NT chains of dependent LDS reads interleaved: every chain's node reads
// issue back to back, then the compares.
template <int NT, int NR>
__device__ __forceinline__ void walk_rows(uint32_t tree, uint32_t rec_bytes, int32_t depth, const uint32_t (&row)[NR],
                                          const uint32_t (&fe)[NR], uint32_t (&lf)[NR][NT]) {
    // a = tree + 4 k for node k; its children sit at 2 a - tree and 4 bytes on
    uint32_t cl[NT], cr[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint32_t root = tree + t * rec_bytes;
        cl[t] = 0u - root;
        cr[t] = 4u - root;
        // opaque to the optimizer, which would otherwise rewrite the select
        // of the two offsets as an add after the compare
        asm volatile("" : "+v"(cl[t]), "+v"(cr[t]));
#pragma unroll
        for (int r = 0; r < NR; ++r) lf[r][t] = root + 4u;
    }
    for (int32_t level = 0; level < depth; ++level) {
        uint32_t w[NR][NT];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) w[r][t] = *(lds_u32*)(uintptr_t)lf[r][t];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t x = __builtin_amdgcn_perm(row[r], fe[r], w[r][t]);
                const bool left = (uint16_t)x < (uint16_t)(w[r][t] >> 16);
                lf[r][t] = 2u * lf[r][t] + (left ? cl[t] : cr[t]);
            }
    }
}

// The same for one row.
template <int NT>
__device__ __forceinline__ void walk(uint32_t tree, uint32_t rec_bytes, int32_t depth, uint32_t row, uint32_t fe,
                                     uint32_t (&lf)[NT]) {
    const uint32_t rows[1] = {row}, fes[1] = {fe};
    uint32_t l[1][NT];
    walk_rows<NT, 1>(tree, rec_bytes, depth, rows, fes, l);
#pragma unroll
    for (int t = 0; t < NT; ++t) lf[t] = l[0][t];
}

}  // namespace
}  // namespace tl
