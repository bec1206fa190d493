// Stage 1: KV usage and batch-size projection (Sec. 4.2, Eq. 1-2) with FIFO
// admission of queued requests under the KV check of Sec. 4.3.2.
//
// One workgroup of one or four wavefronts per scenario (launch_project chooses);
// the per-iteration curves live in LDS.
//
// In-flight requests are turned into O(1) events each instead of O(r) curve
// updates.  For a request with c cached tokens active on [0, e):
//   KV_i[j] = ceil((c + j) / N)   (Eq. 1 with j - s_i = g_i + j)
// starts at ceil(c / N), grows by one block at every j >= 1 with
// c + j == 1 (mod N) -- a comb of period N -- and drops to 0 at e.  An array
// X whose stride-N prefix sums are the curve's differences takes +1 / -1 at the
// comb's ends and, for a jump of v at p, +v at p and -v at p + N; a stride-N
// and a plain prefix sum, in place, give KV.  The batch curve is the prefix sum
// of +1 at 0 / -1 at e.  Every request is read once.
//
// For admission control a new query can be appended to every scenario as a
// request that starts now (Sec. 4.3.2, the "virtual" scoreboard); it adds
// in-flight events like the others.
//
// Queued requests are admitted in FIFO order by the same workgroup, each at the
// first iteration from its arrival (and from the previous admission) where
// its KV contribution over its in-horizon lifetime fits under the capacity.
// Admissions only happen after the last iteration at which the in-flight
// batch alone exceeds the capacity, which makes the lifetime check equal to
// checking the whole projected vector from the current iteration on.
// Without a batch cap the whole queue is tried at its FIFO targets first,
// with O(1) events per request and one check of the summed curve (boards whose
// capacity never binds are done then), else a leading part of it that fits;
// past that, where the capacity binds, the requests that the head's start has
// room for are admitted together.
#include "device_util.h"
#include "queue_tries.h"
#include "tl_internal.h"

namespace tl {
namespace {

constexpr uint64_t kNoDeadline = ~0ull;

__device__ __forceinline__ bool entry_ok(int32_t p, int32_t g, int32_t r, int32_t a) {
    return p >= 0 && g >= 0 && r >= 1 && a >= -1 && (int64_t)p + (int64_t)g <= (1ll << 30);
}

// sum of DA[t] for t in (j, j2], j2 < H; every lane returns the same value
__device__ __forceinline__ int32_t sum_range(const int32_t* DA, int32_t j, int32_t j2) {
    if (j2 == j + 1) return __builtin_amdgcn_readfirstlane(DA[j2]);
    int32_t acc = 0;
    for (int32_t t0 = j + 1; t0 <= j2; t0 += kWave) {
        int32_t t = t0 + lane_id();
        acc += (t <= j2) ? DA[t] : 0;
    }
    return wave_sum(acc);
}

// One workgroup of W (1 or kProjWaves) wavefronts projects a scenario; what
// its wavefronts tell each other.
constexpr int kProjWaves = 4;

struct ProjShared {
    uint64_t u64[kProjWaves];
    int32_t i32[4][kProjWaves];
    uint32_t flag[2];
};

// Waits until this wavefront's global stores and atomics have reached the L2
// cache, where all of its workgroup's are ordered; a barrier after it makes
// them precede the other wavefronts' later ones.  (A device-scope fence also
// writes the whole L2 back: 1024 boards took 190 us with two of them.)
__device__ __forceinline__ void global_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A barrier between accesses to the curves in LDS; one wavefront's are
// processed in order and need none.
template <int W>
__device__ __forceinline__ void curves_sync() {
    if (W > 1) __syncthreads();
    else asm volatile("" ::: "memory");
}

// Whether the condition holds on some thread of the workgroup.  `turn`
// alternates between two flags: one is cleared while the other is in use, and
// the caller has a barrier between a call and the next.
template <int W>
__device__ __forceinline__ bool any_thread(ProjShared& sh, int& turn, bool c) {
    if (W == 1) return __ballot(c) != 0;
    if (__ballot(c) != 0 && lane_id() == 0) sh.flag[turn] = 1;
    __syncthreads();
    const bool r = sh.flag[turn] != 0;
    turn ^= 1;
    if (threadIdx.x == 0) sh.flag[turn] = 0;
    return r;
}

// Adds (or, NEG, takes away) the KV blocks ceil((c + t - a) / N) of a request
// with c cached tokens that starts at iteration a (Eq. 1) to KV[t] for every
// t in [a, lim), a <= lim <= H, 64 iterations per step, by LDS adds that
// return nothing; wavefront w of n takes steps w, w + n, ...
// POW2: N is a power of two no larger than 64 (log2 N = divN.l), so the
// division is a shift and the value grows by exactly 64 / N from one step to
// the next.
template <bool NEG, bool POW2>
__device__ __forceinline__ void add_request(int32_t* KV, int32_t c, int32_t a, int32_t lim, const DivU32& divN,
                                            int w, int n) {
    const int32_t lane = lane_id();
    if (POW2) {
        const int32_t whole = (int32_t)((uint32_t)(lim - a) / kWave);
        int32_t v = (int32_t)(((uint32_t)c + divN.d - 1u + (uint32_t)(w * kWave + lane)) >> divN.l);
        if (NEG) v = -v;
        const int32_t step = (NEG ? -n : n) * (kWave >> divN.l);
        int32_t* q = KV + a + w * kWave + lane;
        int32_t k = w;
        for (; k + 7 * n < whole; k += 8 * n) {
#pragma unroll
            for (int u = 0; u < 8; ++u) atomicAdd(q + u * n * kWave, v + u * step);
            q += 8 * n * kWave;
            v += 8 * step;
        }
        for (; k < whole; k += n) {
            atomicAdd(q, v);
            q += n * kWave;
            v += step;
        }
        if (k == whole && lane < ((lim - a) & (kWave - 1))) atomicAdd(q, v);
    } else {
        for (int32_t t = a + w * kWave + lane; t < lim; t += n * kWave) {
            const int32_t v = (int32_t)ceil_div_u32((uint32_t)(c + t - a), divN);
            atomicAdd(&KV[t], NEG ? -v : v);
        }
    }
}

// The scans below are a workgroup's: its wavefronts take consecutive runs of
// whole 64-iteration steps.  They begin and end with a barrier.
struct ScanRun {
    int32_t from, to;
};
template <int W>
__device__ __forceinline__ ScanRun scan_run(int32_t H, int w) {
    const int32_t per = (H + W * kWave - 1) / (W * kWave) * kWave;
    return ScanRun{min(w * per, H), min((w + 1) * per, H)};
}

// The stride-N prefix sums of X[0 .. H), in place: X[t] += X[t - N] (already
// summed).
template <int W, bool POW2>
__device__ __forceinline__ void strided_scan(int32_t* X, int32_t H, int32_t N) {
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    curves_sync<W>();
    // POW2: N divides 64, so a lane keeps its residue; each wavefront sums its
    // own run, then adds the last sums of the runs before it.  Otherwise one
    // wavefront does it all.
    const ScanRun r = POW2 ? scan_run<W>(H, w) : ScanRun{0, w == 0 ? H : 0};
    const int32_t lane_mod = lane % N;
    for (int32_t t0 = r.from; t0 < r.to; t0 += kWave) {
        const int32_t t = t0 + lane;
        const bool in = t < r.to;
        int32_t c = in ? X[t] : 0;
        for (int32_t d = N; d < kWave; d <<= 1) {
            const int32_t u = __shfl_up(c, d);
            if (lane >= d) c += u;
        }
        const int32_t prev = t0 + lane_mod - N;
        if (prev >= r.from && in) c += X[prev];
        if (in) X[t] = c;
    }
    curves_sync<W>();
    if (POW2 && W > 1) {
        int32_t carry = 0;
        for (int v = 0; v < w; ++v) {
            const ScanRun q = scan_run<W>(H, v);
            // (runs before one that is not empty are whole)
            if (r.from < r.to) carry += X[q.to - N + lane_mod];
        }
        curves_sync<W>();
        for (int32_t t = r.from + lane; t < r.to; t += kWave) X[t] += carry;
        curves_sync<W>();
    }
}

// The prefix sums of X[0 .. H), in place; the last iteration whose sum
// exceeds cap (-1: none), and the first such one from `from` on (H: none).
template <int W>
__device__ __forceinline__ int32_t prefix_scan(ProjShared& sh, int32_t* X, int32_t H, int32_t cap, int32_t from,
                                               int32_t* first_over) {
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    const ScanRun r = scan_run<W>(H, w);
    curves_sync<W>();
    if (W > 1) {
        int32_t sum = 0;
        for (int32_t t = r.from + lane; t < r.to; t += kWave) sum += X[t];
        sum = wave_sum(sum);
        if (lane == 0) sh.i32[0][w] = sum;
        curves_sync<W>();
    }
    int32_t carry = 0, last_over = -1, first = H;
    for (int v = 0; v < w; ++v) carry += sh.i32[0][v];
    for (int32_t t0 = r.from; t0 < r.to; t0 += kWave) {
        const int32_t t = t0 + lane;
        const bool in = t < r.to;
        const int32_t y = wave_incl_scan(in ? X[t] : 0) + carry;
        carry = __builtin_amdgcn_readlane(y, kWave - 1);
        if (in) {
            X[t] = y;
            if (y > cap) {
                last_over = t;
                if (t >= from) first = min(first, t);
            }
        }
    }
    last_over = wave_max(last_over);
    first = H - wave_max(H - first);
    if (W == 1) {
        curves_sync<W>();
        *first_over = first;
        return last_over;
    }
    if (lane == 0) {
        sh.i32[1][w] = last_over;
        sh.i32[2][w] = first;
    }
    curves_sync<W>();
    last_over = -1;
    first = H;
    for (int v = 0; v < W; ++v) {
        last_over = max(last_over, sh.i32[1][v]);
        first = min(first, sh.i32[2][v]);
    }
    *first_over = first;
    return last_over;
}

// Undoes prefix_scan and strided_scan, in place: X[t] -= X[t - 1], then
// X[t] -= X[t - N] of those differences.  From the last iteration down, so
// that every read comes before the write of what it reads.
template <int W>
__device__ __forceinline__ void unscan(int32_t* X, int32_t H, int32_t N) {
    constexpr int kU = 4, kThreads = W * kWave;
    for (int32_t t1 = (H + kU * kThreads - 1) / (kU * kThreads) * (kU * kThreads); t1 > 0;
         t1 -= kU * kThreads) {
        curves_sync<W>();
        int32_t v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t t = t1 - (u + 1) * kThreads + (int32_t)threadIdx.x;
            v[u] = 0;
            if (t < H) {
                v[u] = X[t];
                if (t >= 1) v[u] -= X[t - 1];
                if (t >= N) v[u] -= X[t - N];
                if (t > N) v[u] += X[t - N - 1];
            }
        }
        curves_sync<W>();
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t t = t1 - (u + 1) * kThreads + (int32_t)threadIdx.x;
            if (t < H) X[t] = v[u];
        }
    }
    curves_sync<W>();
}

// Events of a request with c cached tokens in the batch on [a, e), a < H, in
// an array whose stride-N prefix sums' prefix sums are the KV curve: sign times
// its KV blocks ceil((c + t - a) / N).  A jump of v at p is +v at p and -v at
// p + N; the comb of its new blocks starts at its first new-block iteration and
// stops at the first comb point past its end.  START: with the jump at a.
template <bool START>
__device__ __forceinline__ void add_events(int32_t* X, int32_t c, int32_t a, int64_t e, int32_t H, int32_t N,
                                           const DivU32& divN, int32_t sign) {
    if (START) {
        const int32_t v = (int32_t)ceil_div_u32((uint32_t)c, divN);
        atomicAdd(&X[a], sign * v);
        if (N < H - a) atomicAdd(&X[a + N], -sign * v);
    }
    const int32_t rc = (int32_t)((uint32_t)c - div_u32((uint32_t)c, divN) * (uint32_t)N);
    const int64_t j0 = (int64_t)a + (rc == 0 ? 1 : N + 1 - rc);
    if (j0 < min(e, (int64_t)H)) {
        atomicAdd(&X[j0], sign);
        if (e < H) {
            const int64_t jend = j0 + (int64_t)N * (int32_t)ceil_div_u32((uint32_t)(e - j0), divN);
            if (jend < H) atomicAdd(&X[jend], -sign);
        }
    }
    if (e < H) {
        const int32_t w = (int32_t)ceil_div_u32((uint32_t)(c + (int32_t)(e - a) - 1), divN);
        atomicAdd(&X[e], -sign * w);
        if (e + N < H) atomicAdd(&X[e + N], sign * w);
    }
}

// Adds (or takes away) the contributions of the chunk's requests in `take`,
// request m starting at a (its own lane's) and ending, in the horizon, at
// lim: whole requests to the wavefronts in turn.  *r_end: the last end.
template <int W, bool NEG, bool POW2>
__device__ __forceinline__ void add_members(int32_t* KV, uint64_t take, int32_t c, int32_t a, int32_t lim,
                                            const DivU32& divN, int wave, int32_t* r_end) {
    int32_t end = 0;
    int i = 0;
    for (uint64_t mm = take; mm; mm &= mm - 1, ++i) {
        const int m = __ffsll((unsigned long long)mm) - 1;
        const int32_t l = __builtin_amdgcn_readlane(lim, m);
        end = max(end, l);
        if (i % W == wave)
            add_request<NEG, POW2>(KV, __builtin_amdgcn_readlane(c, m), __builtin_amdgcn_readlane(a, m), l, divN, 0, 1);
    }
    *r_end = end;
}

// After such additions: whether KV stays within cap on [from, to).  Every
// wavefront checks a part; a barrier before and one after.
template <int W>
__device__ __forceinline__ bool members_fit(ProjShared& sh, int& turn, const int32_t* KV, int32_t from, int32_t to,
                                            int32_t cap) {
    curves_sync<W>();
    bool over = false;
    if (cap != INT32_MAX)
        for (int32_t t0 = from; t0 < to; t0 += 4 * W * kWave) {
            int32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = KV[min(t0 + u * W * kWave + (int32_t)threadIdx.x, to - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) over |= v[u] > cap;
        }
    return !any_thread<W>(sh, turn, over);
}

// Scenario order for long FIFO loops: a scenario's time grows with its number
// of requests; launched heaviest first, the last workgroups of the grid are
// short ones instead of whichever came last.  A
// counting sort over kOrderBuckets classes of the request count (six per
// doubling), heaviest class first; the order inside a class is whatever the
// atomics give (each scenario's results do not depend on it).  Workspace:
// the counters, then the order [S].
constexpr int kOrderBuckets = 128;

__device__ __forceinline__ int order_bucket(const int64_t* off, int64_t s) {
    const int64_t n = off[s + 1] - off[s];
    const float c = n > 0 ? (float)n : 0.0f;   // malformed offsets: lightest class
    return kOrderBuckets - 1 - min(kOrderBuckets - 1, (int)(log2f(c + 1.0f) * 6.0f));
}

__global__ __launch_bounds__(kOrderBuckets) void order_clear_kernel(uint32_t* counts) {
    counts[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void order_count_kernel(const int64_t* off, int64_t S, uint32_t* counts) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s < S) atomicAdd(&counts[order_bucket(off, s)], 1u);
}

// exclusive prefix of the class counts, in place: each becomes its class's
// first position
__global__ __launch_bounds__(kWave) void order_start_kernel(uint32_t* counts) {
    uint32_t carry = 0;
    for (int i0 = 0; i0 < kOrderBuckets; i0 += kWave) {
        const uint32_t c = counts[i0 + lane_id()];
        const uint32_t incl = (uint32_t)wave_incl_scan((int32_t)c) + carry;
        counts[i0 + lane_id()] = incl - c;
        carry = (uint32_t)__builtin_amdgcn_readlane((int32_t)incl, kWave - 1);
    }
}

__global__ __launch_bounds__(256) void order_place_kernel(const int64_t* off, int64_t S, uint32_t* counts,
                                                          int32_t* order) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s < S) order[atomicAdd(&counts[order_bucket(off, s)], 1u)] = (int32_t)s;
}

constexpr size_t kLdsPerCu = 160 * 1024;

// BD_LDS: the batch difference array lives in LDS beside the KV curve, as a
// batch cap needs (the admission loop reads its running sums).  Without a
// cap it is only added to and finally prefix-summed, so it accumulates with
// atomics in the scenario's own batch output row instead: half the LDS, twice
// the scenario wavefronts per CU.
// CAP: with a batch cap.  A constant, so that neither kind of loop carries the
// other's state (both in one kernel: 102 scalar registers spilled behind a cap,
// each spill and reload an instruction in a chain bound by its latency; now
// none).
// W wavefronts a scenario, A (1 or W) of them in the admission loop.
template <bool CAP, bool BD_LDS, bool POW2, int W, int A>
__global__ __launch_bounds__(W* kWave) void project_kernel(ProjectParams P) {
    static_assert(BD_LDS || !CAP, "a batch cap reads running sums of the batch differences");
    extern __shared__ int32_t lds[];
    __shared__ ProjShared sh;
    const int32_t H = P.H;
    const int32_t N = P.N;
    const DivU32 divN{(uint32_t)N, P.div_m, P.div_l};
    const int lane = lane_id();
    const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t block = P.first_block + blockIdx.x;
    const int64_t s = P.order_ws ? (int64_t)((const int32_t*)P.order_ws + kOrderBuckets)[block] : block;
    int32_t* outB = P.batch + s * H;
    int32_t* KV = lds;                      // events, then KV values
    int32_t* BI = BD_LDS ? lds + H : outB;  // batch difference array
    int32_t* outKV = P.kv + s * H;
    uint64_t* outDL = P.deadline_at + s * H;

    for (int32_t t = threadIdx.x; t < H; t += W * kWave) {
        KV[t] = 0;
        BI[t] = 0;
        outDL[t] = kNoDeadline;
    }
    if (threadIdx.x < 2) sh.flag[threadIdx.x] = 0;
    int turn = 0;
    global_done();
    __syncthreads();

    const int64_t lo = P.off[s];
    const int64_t hi = P.off[s + 1];
    const bool bad_range = lo < 0 || hi < lo || hi > P.n_requests || hi - lo > 0x7fffffffll;

    // Every request once, each wavefront a run of them: validity, size guard,
    // lost / queue information; the in-flight ones' KV events (the jumps at
    // iteration 0 summed in registers), batch events and deadlines.
    uint64_t bound = 0;
    uint32_t fl = 0;
    int32_t has_queue = 0, n_end = 0, n_in = 0, kv0 = 0;
    int32_t arr_max = -1, arr_min = INT32_MAX;   // of the run's queued arrivals
    if (!bad_range) {
        const int64_t per = (hi - lo + W * kWave - 1) / (W * kWave) * kWave;
        const int64_t r0 = lo + wave * per, r1 = min(r0 + per, hi);
        for (int64_t base = r0; base < r1; base += kWave) {
            const int64_t i = base + lane;
            const bool in = i < r1;
            int32_t p = 0, g = 0, r = 0, a = -1;
            uint64_t d = kNoDeadline;
            bool is_lost = false;
            if (in) {
                p = P.prompt[i];
                g = P.gen[i];
                r = P.rem[i];
                a = P.arr[i];
                if (P.lost) is_lost = P.lost[i] != 0;
                if (P.deadline) d = P.deadline[i];
            }
            const bool ok = in && entry_ok(p, g, r, a);
            if (in && !ok) fl |= TL_FLAG_BAD_REQUEST;
            if (ok) bound += ceil_div_u32((uint32_t)(p + g + H), divN);
            if (ok && a == -1) {
                if (is_lost) fl |= TL_FLAG_LOST;
                ++n_in;
                kv0 += (int32_t)ceil_div_u32((uint32_t)(p + g), divN);
                n_end = max(n_end, min(r, H));
                add_events<false>(KV, p + g, 0, r, H, N, divN, 1);
                if (r < H) atomicAdd(&BI[r], -1);
                if (r <= H && !is_lost && d != kNoDeadline)
                    atomicMin((unsigned long long*)&outDL[r - 1], (unsigned long long)d);
            }
            const bool queued = ok && a >= 0;
            if (__ballot(queued)) {
                if (queued && a < H) has_queue = 1;
                // queue order: each queued arrival must be >= every earlier one
                const int32_t incl = wave_incl_max(queued ? a : -1);
                const int32_t excl = max(wave_shift_up1(incl, -1), arr_max);
                if (queued && a < excl) fl |= TL_FLAG_UNSORTED;
                arr_max = max(arr_max, lane63(incl));
                if (queued) arr_min = min(arr_min, a);
            }
        }
    }
    // the appended query (admission control): one more request that starts
    // now; a malformed one is left out and flagged
    if (P.cand_len && !bad_range) {
        const int32_t cand_p = P.cand_prompt[s];
        const int32_t cand_l = P.cand_len[s];
        if (!entry_ok(cand_p, 0, cand_l, -1)) {
            fl |= TL_FLAG_BAD_CANDIDATE;
        } else if (threadIdx.x == 0) {
            bound += ceil_div_u32((uint32_t)(cand_p + H), divN);
            ++n_in;
            kv0 += (int32_t)ceil_div_u32((uint32_t)cand_p, divN);
            n_end = max(n_end, min(cand_l, H));
            add_events<false>(KV, cand_p, 0, cand_l, H, N, divN, 1);
            if (cand_l < H) atomicAdd(&BI[cand_l], -1);
        }
    }
    // over the wavefronts; a run's arrivals below an earlier run's largest
    // are out of order too
    bound = wave_sum_u64(bound);
    fl = wave_or(fl) | (wave_max(has_queue) ? 1u << 31 : 0u);
    arr_min = INT32_MAX - wave_max(INT32_MAX - arr_min);
    n_end = wave_max(n_end);
    n_in = wave_sum(n_in);
    kv0 = wave_sum(kv0);
    // (every atomic on the outputs is done before another wavefront goes on)
    global_done();
    if (lane == 0) {
        sh.u64[wave] = bound;
        sh.i32[0][wave] = (int32_t)fl;
        sh.i32[1][wave] = n_end;
        sh.i32[2][wave] = arr_min;
        sh.i32[3][wave] = arr_max;
        if (n_in) atomicAdd(&BI[0], n_in);
        if (kv0) {
            atomicAdd(&KV[0], kv0);
            if (N < H) atomicAdd(&KV[N], -kv0);
        }
    }
    __syncthreads();
    bound = 0;
    fl = 0;
    n_end = 0;
    arr_max = -1;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        bound += sh.u64[w];
        fl |= (uint32_t)sh.i32[0][w];
        n_end = max(n_end, sh.i32[1][w]);
        if (sh.i32[2][w] < arr_max) fl |= TL_FLAG_UNSORTED;
        arr_max = max(arr_max, sh.i32[3][w]);
    }
    // (wavefront-uniform, like everything the admission loop decides on)
    fl = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)fl);
    n_end = __builtin_amdgcn_readfirstlane(n_end);
    bound = lane63_u64(bound);
    const bool has_queue_any = (fl >> 31) != 0;
    fl &= ~(1u << 31);

    if (bad_range || bound > 0x7fffffffull) {
        for (int32_t t = threadIdx.x; t < H; t += W * kWave) {
            outB[t] = 0;
            outKV[t] = 0;
            outDL[t] = kNoDeadline;
        }
        if (threadIdx.x == 0) {
            P.n_iters[s] = 0;
            P.flags[s] = bad_range ? TL_FLAG_OVERFLOW : ((fl & TL_FLAG_BAD_REQUEST) | TL_FLAG_OVERFLOW);
        }
        return;
    }

    // the KV curve; last over-capacity iteration.  The batch curve stays
    // a difference array: admissions add their +1 / -1 to it and the output
    // takes its prefix sum.
    const int32_t cap = P.kv_cap[s];
    // bound is at least the KV of every iteration: when it fits the
    // capacity, no admission check can fail and the checks are skipped
    const bool kv_fits = cap >= 0 && bound <= (uint64_t)cap;
    int32_t first_over = H;   // (of the whole queue's sum, below)
    strided_scan<W, POW2>(KV, H, N);
    const int32_t last_over = __builtin_amdgcn_readfirstlane(prefix_scan<W>(sh, KV, H, cap, 0, &first_over));
    const int32_t bcap = CAP ? P.batch_cap[s] : 0;
    if (last_over >= 0 || (CAP && __builtin_amdgcn_readfirstlane(BI[0]) > bcap)) fl |= TL_FLAG_OVERCOMMIT;

    // FIFO admission of queued requests.  Every wavefront takes part in the tries
    // of the whole queue; the loop over the rest is run by A wavefronts, the
    // others wait.  The values it carries (iteration j, batch size, the head's
    // fields, check outcomes) are the same in all A, wavefront-uniform and kept in
    // scalar registers.  They come from reads of the curves between barriers;
    // the additions to the curves and the checks over many iterations are
    // shared out, and wavefront 0 alone writes the batch events and deadlines.
    int32_t* BD = BI;   // batch differences: in-flight requests, then admitted ones
    if (has_queue_any) {
        curves_sync<W>();
        int32_t j = 0;
        int32_t run = 0;    // batch size at j (prefix of BD; kept only under a batch cap)
        if (CAP) run = __builtin_amdgcn_readfirstlane(BD[0]);
        // (no batch cap) how the next requests are tried, see below
        bool at_targets = true;
        bool alone = false;
        int32_t fmax = kWave;          // requests tried at one start at most
        int32_t calm = 0, calm_need = 4;
        int32_t streak = 0, streak_need = 0;
        int64_t cb = lo - kWave;
        int32_t q_arr = 0, q_c = 0, q_len = 0, q_lost = 0;
        // (no batch cap) running maximum of the chunk's arrivals, the blocks
        // a request starts with, and their running sum
        int32_t q_max = -1, q_c0 = 0, q_sum = 0;
        uint64_t q_dl = kNoDeadline;
        uint64_t mask = 0;
        bool whole = !CAP && hi - lo >= 2 * kWave;
        for (;;) {
            if (whole) {
                // All remaining requests at once, each at its FIFO target (the
                // running maximum of the arrivals, from max(j, last_over +
                // 1)): O(1) events a request, one scan, one check.  When the
                // sum fits everywhere, so does every request's own check at
                // its target (each sees the KV of the requests before it, which
                // is no more than the sum): these are the admissions that the
                // one-at-a-time loop makes.  Otherwise some leading chunks of 64
                // requests that fit together: the chunks that have arrived when
                // the whole sum first exceeds the capacity (without later
                // arrivals it falls from there), and the like (QueueTries).
                const int64_t first = cb + kWave;
                const int32_t n_ch = (int32_t)((hi - first + kWave - 1) / kWave);
                const int32_t lo_j = max(j, last_over + 1);
                // Chunks from .. to - 1, a run of them per wavefront: their
                // events times sign, or (commit) their batch events, deadlines
                // and n_end.
                auto run_before = [&](int32_t k) {   // running maximum of the targets before chunk k
                    int32_t m = lo_j;
                    if (fl & TL_FLAG_UNSORTED) {
                        for (int64_t i = first + lane; i < min(first + (int64_t)k * kWave, hi); i += kWave) {
                            const int32_t a = P.arr[i];
                            if (a > m && entry_ok(P.prompt[i], P.gen[i], P.rem[i], a)) m = a;
                        }
                        return wave_max(m);
                    }
                    // sorted: the last valid queued entry before the chunk
                    for (int64_t i1 = first + (int64_t)k * kWave; i1 > first; i1 -= kWave) {
                        const int64_t i = i1 - kWave + lane;
                        const int32_t a = i < hi ? P.arr[i] : -1;
                        const bool q = a >= 0 && entry_ok(P.prompt[i], P.gen[i], P.rem[i], a);
                        if (__ballot(q)) return max(m, wave_max(q ? a : -1));
                    }
                    return m;
                };
                auto chunks = [&](int32_t from, int32_t to, int32_t sign, bool commit) {
                    // each wavefront a run of chunks
                    const int32_t per = (to - from + W - 1) / W;
                    const int32_t k0 = min(from + wave * per, to), k1 = min(k0 + per, to);
                    if (k0 >= k1) return;
                    int32_t run = run_before(k0);
                    // the next chunk's fields are fetched while one is worked on
                    int32_t na = -1, np = 0, ng = 0, nr = 0;
                    auto fetch = [&](int32_t k) {
                        const int64_t i = first + (int64_t)k * kWave + lane;
                        na = -1;
                        if (k < k1 && i < hi) {
                            na = P.arr[i];
                            np = P.prompt[i];
                            ng = P.gen[i];
                            nr = P.rem[i];
                        }
                    };
                    fetch(k0);
                    for (int32_t k = k0; k < k1; ++k) {
                        const int64_t i = first + (int64_t)k * kWave + lane;
                        int32_t a = na;
                        const int32_t c = np + ng, len = nr;
                        const bool q = a >= 0 && entry_ok(np, ng, nr, a);
                        fetch(k + 1);
                        a = max(wave_incl_max(q ? a : -1), run);
                        run = __builtin_amdgcn_readlane(a, kWave - 1);
                        if (q && a < H) {
                            const int64_t e = (int64_t)a + len;
                            if (!commit) {
                                add_events<true>(KV, c, a, e, H, N, divN, sign);
                            } else {
                                atomicAdd(&BD[a], 1);
                                if (e < H) atomicAdd(&BD[e], -1);
                                const uint64_t dl = P.deadline ? P.deadline[i] : kNoDeadline;
                                if (e <= H && dl != kNoDeadline && !(P.lost && P.lost[i]))
                                    atomicMin((unsigned long long*)&outDL[e - 1], (unsigned long long)dl);
                                n_end = max(n_end, (int32_t)min(e, (int64_t)H));
                            }
                        }
                    }
                };
                QueueTries t(n_ch);
                int32_t cur = 0;
                for (;;) {
                    unscan<W>(KV, H, N);
                    if (t.want > cur) chunks(cur, t.want, 1, false);
                    else chunks(t.want, cur, -1, false);
                    strided_scan<W, POW2>(KV, H, N);
                    const bool fits = prefix_scan<W>(sh, KV, H, cap, last_over + 1, &first_over) <= last_over || kv_fits;
                    cur = t.want;
                    int32_t guess = -1;
                    if (!fits && cur == n_ch) {
                        for (int32_t k0 = 0; k0 < n_ch; k0 += kWave) {
                            const int32_t k = k0 + lane;
                            const int32_t a = k < n_ch ? P.arr[first + (int64_t)k * kWave] : INT32_MAX;
                            guess += (int32_t)__builtin_popcountll(__ballot(a <= first_over));
                        }
                    }
                    if (!t.after(fits, guess)) break;
                }
                const int32_t ok = t.ok;
                if (ok > 0) {
                    chunks(0, ok, 1, true);
                    n_end = wave_max(n_end);
                    curves_sync<W>();
                    if (lane == 0) sh.i32[0][wave] = n_end;
                    curves_sync<W>();
                    for (int w = 0; w < W; ++w) n_end = max(n_end, sh.i32[0][w]);
                    n_end = __builtin_amdgcn_readfirstlane(n_end);
                    const int32_t run = run_before(ok);
                    if (run >= H) break;   // the head cannot start within the horizon
                    j = run;
                }
                cb += (int64_t)ok * kWave;
                streak = 0;
                if (ok < n_ch) {
                    streak_need = min(64, max(4, 2 * streak_need));
                    at_targets = false;
                    calm = 0;
                }
            }
            bool again = false;
            if (A == W || wave == 0) {
                for (;;) {
                    if (!CAP && mask == 0 && streak >= streak_need && hi - (cb + kWave) >= 2 * kWave) {
                        again = true;
                        break;
                    }
                    while (mask == 0) {
                        cb += kWave;
                        if (cb >= hi) break;
                        const int64_t i = cb + lane;
                        bool q = false;
                        if (i < hi) {
                            q_arr = P.arr[i];
                            const int32_t p = P.prompt[i], g = P.gen[i];
                            q_len = P.rem[i];
                            q = entry_ok(p, g, q_len, q_arr) && q_arr >= 0;
                            q_c = p + g;
                            q_lost = P.lost ? P.lost[i] : 0;
                            q_dl = P.deadline ? P.deadline[i] : kNoDeadline;
                        }
                        mask = __ballot(q);
                        if (!CAP && mask) {
                            q_max = wave_incl_max(q ? q_arr : -1);
                            q_c0 = q ? (int32_t)ceil_div_u32((uint32_t)q_c, divN) : 0;
                            q_sum = wave_incl_scan(q_c0);
                        }
                    }
                    if (mask == 0) break;

                    if (!CAP && at_targets) {
                        // The rest of this chunk of the queue, each at its FIFO
                        // target, as above; their contributions are added to the KV
                        // curve iteration by iteration and taken out again when they
                        // do not fit.
                        const int32_t lo_j = max(j, last_over + 1);
                        const bool mem = (mask >> lane) & 1;
                        const int32_t a = wave_incl_max(mem ? max(q_arr, lo_j) : -1);
                        const uint64_t memm = __ballot(mem);
                        const uint64_t over = __ballot(mem && a >= H);
                        const uint64_t take = over ? (memm & ((over & (~over + 1)) - 1)) : memm;
                        if (take == 0) break;   // the head cannot start within the horizon
                        // each member's in-horizon end, on its own lane
                        const int32_t lim_l = q_len >= H - a ? H : a + q_len;
                        const int32_t a_first = __builtin_amdgcn_readlane(a, __ffsll((unsigned long long)take) - 1);
                        int32_t r_end = 0;
                        add_members<A, false, POW2>(KV, take, q_c, a, lim_l, divN, wave, &r_end);
                        if (!members_fit<A>(sh, turn, KV, a_first, r_end, kv_fits ? INT32_MAX : cap)) {
                            // take the batch's contributions out again
                            add_members<A, true, POW2>(KV, take, q_c, a, lim_l, divN, wave, &r_end);
                            curves_sync<A>();
                            at_targets = false;
                            streak = 0;
                            calm = 0;
                            calm_need = min(256, 2 * calm_need);
                            continue;
                        }
                        if (wave == 0 && ((take >> lane) & 1)) {
                            const int64_t e = (int64_t)a + q_len;
                            atomicAdd(&BD[a], 1);
                            if (e < H) atomicAdd(&BD[e], -1);
                            if (e <= H && !q_lost && q_dl != kNoDeadline)
                                atomicMin((unsigned long long*)&outDL[e - 1], (unsigned long long)q_dl);
                        }
                        n_end = max(n_end, r_end);
                        j = __builtin_amdgcn_readlane(a, 63 - __clzll((long long)take));
                        mask &= ~take;
                        ++streak;
                        if (streak >= 4) calm_need = 4;
                        if (over) break;
                        continue;
                    }

                    if (!CAP && !alone) {
                        // The capacity binds: the head and the requests behind it that
                        // have arrived by its start j, as many as the KV of iteration
                        // j itself leaves room for.  When their sum fits everywhere,
                        // they are the one-at-a-time loop's admissions at j, and the
                        // next of them does not fit at j.  A head without room at j
                        // starts no earlier than the next iteration that has it.
                        const bool queued = (mask >> lane) & 1;
                        const int hl = __ffsll((unsigned long long)mask) - 1;
                        const int32_t start = max(max(j, last_over + 1), __builtin_amdgcn_readlane(q_max, hl));
                        const int32_t c_h = __builtin_amdgcn_readlane(q_c0, hl);
                        int32_t room = -1, found = -1;
                        for (int32_t t0 = start; t0 < H; t0 += kWave) {
                            const int32_t t = t0 + lane;
                            const int32_t left = cap - KV[min(t, H - 1)];
                            const uint64_t m = __ballot(t < H && left >= c_h);
                            if (m) {
                                const int l = __ffsll((unsigned long long)m) - 1;
                                found = t0 + l;
                                room = __builtin_amdgcn_readlane(left, l);
                                break;
                            }
                        }
                        if (found < 0) break;   // the head cannot start within the horizon
                        if (found > start) calm = 0;
                        j = found;
                        // the requests behind it that have arrived (those before it in
                        // the chunk, admitted by now, arrived no later than j)
                        const bool mem = queued && q_max <= j;
                        const int32_t sum = q_sum - (__builtin_amdgcn_readlane(q_sum, hl) - c_h);
                        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                        const uint64_t take = __ballot(mem && sum <= room && (int32_t)below < fmax);
                        const uint64_t blocked = __ballot(mem && sum > room);
                        if ((take & (take - 1)) == 0) {
                            alone = true;   // one request: checked below before it is added
                            continue;
                        }
                        const int32_t lim_l = q_len >= H - j ? H : j + q_len;
                        int32_t r_end = 0;
                        // (everyone has read the curve above before it changes)
                        curves_sync<A>();
                        add_members<A, false, POW2>(KV, take, q_c, j, lim_l, divN, wave, &r_end);
                        if (!members_fit<A>(sh, turn, KV, j, r_end, cap)) {
                            add_members<A, true, POW2>(KV, take, q_c, j, lim_l, divN, wave, &r_end);
                            curves_sync<A>();
                            fmax = max(1, (int32_t)__builtin_popcountll(take) >> 2);
                            calm = 0;
                            continue;
                        }
                        if (wave == 0 && ((take >> lane) & 1)) {
                            const int64_t e = (int64_t)j + q_len;
                            if (e < H) atomicAdd(&BD[e], -1);
                            if (e <= H && !q_lost && q_dl != kNoDeadline)
                                atomicMin((unsigned long long*)&outDL[e - 1], (unsigned long long)q_dl);
                        }
                        if (threadIdx.x == 0) atomicAdd(&BD[j], (int32_t)__builtin_popcountll(take));
                        n_end = max(n_end, r_end);
                        mask &= ~take;
                        fmax = min(kWave, 2 * fmax);
                        calm = blocked ? 0 : calm + 1;
                        if (calm >= calm_need) {
                            at_targets = true;
                            streak = 0;
                        }
                        continue;
                    }

                    // One request at a time (under a batch cap, or one without
                    // company).  The head of the queue: uniform lane, lane reads.
                    const int hl = __ffsll((unsigned long long)mask) - 1;
                    const int32_t h_arr = __builtin_amdgcn_readlane(q_arr, hl);
                    const int32_t h_c = __builtin_amdgcn_readlane(q_c, hl);
                    const int32_t h_len = __builtin_amdgcn_readlane(q_len, hl);
                    const int32_t h_lost = __builtin_amdgcn_readlane(q_lost, hl);
                    const uint64_t h_dl =
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(q_dl >> 32), hl) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)q_dl, hl);
                    const int32_t target = max(max(h_arr, j), last_over + 1);
                    if (h_arr >= H || target >= H) break;
                    if (CAP && target > j) run += sum_range(BD, j, target);
                    j = target;
                    bool admitted = false;
                    for (;;) {
                        bool ok = !CAP || run < bcap;
                        int32_t t_bad = -1;
                        if (ok) {
                            // 4 x 64 iterations per round (their LDS reads in flight
                            // together); the earliest overflowing iteration wins
                            const int32_t lim = kv_fits ? j : (int32_t)min((int64_t)j + h_len, (int64_t)H);
                            for (int32_t t0 = j; t0 < lim && t_bad < 0; t0 += 4 * kWave) {
                                uint64_t m[4];
        #pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const int32_t t = t0 + k * kWave + lane;
                                    bool badt = false;
                                    if (t < lim)
                                        badt = KV[t] + (int32_t)(POW2 ? ((uint32_t)(h_c + t - j) + divN.d - 1u) >> divN.l
                                                                      : ceil_div_u32((uint32_t)(h_c + t - j), divN)) > cap;
                                    m[k] = __ballot(badt);
                                }
        #pragma unroll
                                for (int k = 3; k >= 0; --k)
                                    if (m[k]) t_bad = t0 + k * kWave + __ffsll((unsigned long long)m[k]) - 1;
                            }
                            ok = t_bad < 0;
                        }
                        if (ok) { admitted = true; break; }
                        if (CAP && run >= bcap) {
                            // The batch is full: the next start to try is the first
                            // later iteration with a free slot, found 64 iterations
                            // at a time from the batch differences (what stepping
                            // one iteration at a time reaches).
                            int32_t base = j, r = run, found = -1;
                            while (base + 1 < H) {
                                const int32_t t = base + 1 + lane;
                                const int32_t pre = wave_incl_scan(t < H ? BD[t] : 0) + r;   // batch size at t
                                const uint64_t m = __ballot(t < H && pre < bcap);
                                if (m) {
                                    const int l = __ffsll((unsigned long long)m) - 1;
                                    found = base + 1 + l;
                                    r = __builtin_amdgcn_readlane(pre, l);
                                    break;
                                }
                                r = __builtin_amdgcn_readlane(pre, kWave - 1);
                                base += kWave;
                            }
                            if (found < 0) break;
                            run = r;
                            j = found;
                            continue;
                        }
                        // Next start to try.  If iteration t_bad overflowed, every
                        // start j2 in (j, t_bad] whose own contribution there,
                        // ceil((c + t_bad - j2) / N), exceeds room = cap - KV[t_bad]
                        // fails the same way: j2 < c + t_bad - N * room (all of
                        // them when room < 0).  Skipping those gives the same
                        // admission iteration.
                        int32_t nj = j + 1;
                        if (t_bad >= 0) {
                            const int32_t room = cap - __builtin_amdgcn_readfirstlane(KV[t_bad]);
                            int64_t first = (int64_t)t_bad + 1;
                            if (room >= 0) first = min(first, (int64_t)h_c + t_bad - (int64_t)N * room);
                            nj = (int32_t)max((int64_t)nj, first);
                        }
                        if (nj >= H) break;
                        if (CAP) run += sum_range(BD, j, nj);
                        j = nj;
                    }
                    if (!admitted) break;
                    const int64_t e = (int64_t)j + h_len;
                    const int32_t lim = (int32_t)min(e, (int64_t)H);
                    curves_sync<A>();   // everyone has read the curves
                    add_request<false, POW2>(KV, h_c, j, lim, divN, wave, A);
                    if (threadIdx.x == 0) {
                        if (BD_LDS) {
                            BD[j] += 1;
                            if (e < H) BD[e] -= 1;
                        } else {
                            atomicAdd(&BD[j], 1);
                            if (e < H) atomicAdd(&BD[e], -1);
                        }
                        if (e <= H && !h_lost && h_dl != kNoDeadline)
                            atomicMin((unsigned long long*)&outDL[e - 1], (unsigned long long)h_dl);
                    }
                    run += 1;
                    n_end = max(n_end, lim);
                    mask &= mask - 1;
                    curves_sync<A>();
                    alone = false;
                    fmax = min(kWave, 2 * fmax);
                }
            }
            if (A < W) {   // where the loop has come to
                curves_sync<W>();
                if (threadIdx.x == 0) {
                    sh.u64[0] = (uint64_t)cb;
                    sh.i32[0][0] = again;
                    sh.i32[1][0] = j;
                    sh.i32[2][0] = n_end;
                }
                curves_sync<W>();
                cb = (int64_t)lane63_u64(sh.u64[0]);
                again = __builtin_amdgcn_readfirstlane(sh.i32[0][0]) != 0;
                j = __builtin_amdgcn_readfirstlane(sh.i32[1][0]);
                n_end = __builtin_amdgcn_readfirstlane(sh.i32[2][0]);
            }
            if (!again) break;
            whole = true;
        }
    }
    global_done();
    __syncthreads();

    // outputs: curves (batch = prefix sum of BD), scalars.  Each wavefront a
    // run of iterations: its total, then its sums.  (Differences kept in the
    // output row were added at L2 by atomics: they are read there, eight
    // 64-iteration chunks in flight at a time.)
    const ScanRun run = scan_run<W>(H, wave);
    constexpr int kChunks = 8;
    auto load = [&](int32_t t) {
        return BD_LDS ? BD[t] : __hip_atomic_load(&BD[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    int32_t total = 0;
    for (int32_t g0 = run.from; g0 < run.to; g0 += kChunks * kWave) {
        int32_t d[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int32_t t = g0 + c * kWave + lane;
            d[c] = t < run.to ? load(t) : 0;
        }
#pragma unroll
        for (int c = 0; c < kChunks; ++c) total += d[c];
    }
    total = wave_sum(total);
    if (lane == 0) sh.i32[3][wave] = total;
    __syncthreads();
    int32_t carry_b = 0;
    for (int w = 0; w < wave; ++w) carry_b += sh.i32[3][w];
    for (int32_t g0 = run.from; g0 < run.to; g0 += kChunks * kWave) {
        int32_t d[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int32_t t = g0 + c * kWave + lane;
            d[c] = t < run.to ? load(t) : 0;
        }
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int32_t t = g0 + c * kWave + lane;
            const int32_t b = wave_incl_scan(d[c]) + carry_b;
            carry_b = __builtin_amdgcn_readlane(b, kWave - 1);
            if (t < run.to) {
                outB[t] = b;
                outKV[t] = KV[t];
            }
        }
    }
    if (threadIdx.x == 0) {
        P.n_iters[s] = n_end;
        P.flags[s] = fl;
    }
}

// Feature rows of the grid, written out when requested: row (s, f, j) =
// (freq[f], KV[s][j], B[s][j] [, engine[s]]) from the curves project_kernel
// wrote.  One thread per (s, j) writes its F rows with one 16- or 12-byte
// store each; consecutive threads write consecutive rows of one frequency.
constexpr int kRowsThreads = 256;

template <int NF>
__global__ __launch_bounds__(kRowsThreads) void expand_rows_kernel(ProjectParams P) {
    const int32_t H = P.H;
    const int32_t n_jb = (H + kRowsThreads - 1) / kRowsThreads;
    const uint32_t block = (uint32_t)P.first_block + blockIdx.x;   // (fewer than 2^26 of 256 threads)
    const int64_t s = block / (uint32_t)n_jb;
    const int32_t t = (int32_t)(block % (uint32_t)n_jb) * kRowsThreads + threadIdx.x;
    if (t >= H) return;
    const float kf = (float)P.kv[s * H + t], bf = (float)P.batch[s * H + t];
    const float eng = NF == 4 ? P.engine[s] : 0.0f;
    float* row = P.rows + ((int64_t)s * P.F * H + t) * NF;
    const int64_t f_stride = (int64_t)H * NF;
#pragma unroll 4
    for (int32_t f = 0; f < P.F; ++f) {
        if (NF == 4)
            *(float4*)(row + f * f_stride) = make_float4(P.freqs[f], kf, bf, eng);
        else
            *(float3*)(row + f * f_stride) = make_float3(P.freqs[f], kf, bf);
    }
}

// Remaining-token counts from the predictor's total lengths (Sec. 4.6):
// inflate by num/den (rounded up; den = 0: none), limit to max_tokens, reset
// to max_tokens past an outrun prediction, remaining = max(length - gen, 1);
// malformed entries get 0.  One wavefront per scenario, 64 entries a step.
constexpr int kAdjustWaves = 4;

__global__ __launch_bounds__(kAdjustWaves * kWave) void adjust_kernel(AdjustParams P) {
    const int64_t s = (P.first_block + blockIdx.x) * kAdjustWaves + threadIdx.x / kWave;
    if (s >= P.S) return;
    const int64_t lo = P.off[s], hi = P.off[s + 1];
    if (lo < 0 || hi < lo || hi > P.n_requests) return;
    const uint32_t num = P.num[s], den = P.den[s];
    const int32_t mt = P.max_tokens[s];
    for (int64_t i = lo + lane_id(); i < hi; i += kWave) {
        const int32_t g = P.gen[i], r = P.pred[i];
        int32_t out = 0;
        if (g >= 0 && r >= 1) {
            int64_t len = r;
            if (den > 0) {
                const uint64_t x = (uint64_t)r * num;
                len = (int64_t)min((x + den - 1) / den, (uint64_t)0x7fffffff);
            }
            if (mt >= 1) {
                len = min(len, (int64_t)mt);
                if (g >= len) len = mt;
            }
            out = (int32_t)max(len - g, (int64_t)1);
        }
        P.out[i] = out;
    }
}

}  // namespace

hipError_t launch_adjust(const AdjustParams& p, hipStream_t stream) {
    return launch_parts((p.S + kAdjustWaves - 1) / kAdjustWaves, kAdjustWaves * kWave, [&](dim3 grid, int64_t first) {
        AdjustParams q = p;
        q.first_block = first;
        hipLaunchKernelGGL(adjust_kernel, grid, dim3(kAdjustWaves * kWave), 0, stream, q);
    });
}

// Long FIFO loops: no batch cap and on average 1024 or more requests per
// scenario.
bool long_fifo_loops(const ProjectParams& p) {
    return p.batch_cap == nullptr && p.n_requests >= (int64_t)1024 * p.n_scenarios;
}

size_t project_order_bytes(const ProjectParams& p) {
    if (!long_fifo_loops(p) || p.n_scenarios < 2 || p.n_scenarios > 0x7fffffffll) return 0;
    return (size_t)(kOrderBuckets + p.n_scenarios) * sizeof(int32_t);
}

hipError_t launch_project(const ProjectParams& p, hipStream_t stream) {
    // The batch differences go to global memory where occupancy pays (long
    // FIFO loops); otherwise the LDS array is faster.
    const bool bd_lds = !long_fifo_loops(p);
    const size_t lds = (size_t)(bd_lds ? 2 : 1) * p.H * sizeof(int32_t);
    // block sizes that are powers of two up to 64 take shifts instead of
    // divisions in the admission loops
    const bool pow2 = p.N <= kWave && (p.N & (p.N - 1)) == 0;
    // Wavefronts a scenario.  Without a batch cap four share its request pass,
    // scans and tries of the whole queue (us at one / four: 1024 boards in flight
    // 28 / 14, one board x 2048 iterations 23 / 10, 1024 x 1024 with 800 queued and
    // capacity to spare 62 / 38) where the device holds all boards at four each
    // (five a CU with the registers they take), or where the LDS of a board
    // leaves a CU few of them anyway.  Beyond, one: boards whose capacity binds
    // spend their time in the loop, where four bring little and take the place of
    // other boards (2048 x 1024 with 200 queued 482 / 760, 4096 under arrivals
    // 4060 / 8172; 4096 x 3072 with 300 queued 2485 / 2624, with capacity to
    // spare 269 / 156).
    // Of four, one runs the loop and the others wait: with a barrier per
    // admission 1024 x 1024 with 200 queued took 550 us instead of 409, with 1500
    // on 2048 iterations 1116 instead of 880.  All four run it (they share the
    // additions) while every board has a CU to itself (64 x 4096 with 400 queued
    // one 641, four 608; 64 under arrivals 3439 / 3215).
    // Behind a batch cap requests are admitted one at a time, a barrier each
    // between four wavefronts: four only while every board has a CU to itself and
    // its horizon is long enough for them to gain on the additions (us at 1 /
    // 4, 256 boards x 4096 iterations 319 / 262, where the KV capacity binds 536 /
    // 525; 2 x 666 96 / 89, 144 / 140; 1 x 512 61 / 59, 81 / 81; 268 x 302 92 /
    // 97, 119 / 132; 1024 x 4096 337 / 348, 547 / 758; 4096 x 1024 220 / 571).
    const bool cap = p.batch_cap != nullptr;
    constexpr int64_t kCus = 256;
    const bool four = cap ? p.n_scenarios <= kCus && p.H >= 512
                          : p.n_scenarios <= 5 * kCus || lds > kLdsPerCu / 7;
    const int w = four ? kProjWaves : 1;
    const bool all = p.n_scenarios <= kCus;
    constexpr int W = kProjWaves;
    void (*const capped[2][2])(ProjectParams) = {
        {project_kernel<true, true, false, 1, 1>, project_kernel<true, true, false, W, W>},
        {project_kernel<true, true, true, 1, 1>, project_kernel<true, true, true, W, W>}};
    void (*const uncapped[2][2][3])(ProjectParams) = {
        {{project_kernel<false, false, false, 1, 1>, project_kernel<false, false, false, W, 1>,
          project_kernel<false, false, false, W, W>},
         {project_kernel<false, false, true, 1, 1>, project_kernel<false, false, true, W, 1>,
          project_kernel<false, false, true, W, W>}},
        {{project_kernel<false, true, false, 1, 1>, project_kernel<false, true, false, W, 1>,
          project_kernel<false, true, false, W, W>},
         {project_kernel<false, true, true, 1, 1>, project_kernel<false, true, true, W, 1>,
          project_kernel<false, true, true, W, W>}}};
    void (*const kern)(ProjectParams) = cap ? capped[pow2][four] : uncapped[bd_lds][pow2][four ? 1 + all : 0];
    if (lds + sizeof(ProjShared) > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (p.order_ws) {
        uint32_t* counts = (uint32_t*)p.order_ws;
        const unsigned nb = (unsigned)((p.n_scenarios + 255) / 256);
        hipLaunchKernelGGL(order_clear_kernel, dim3(1), dim3(kOrderBuckets), 0, stream, counts);
        hipLaunchKernelGGL(order_count_kernel, dim3(nb), dim3(256), 0, stream, p.off, p.n_scenarios, counts);
        hipLaunchKernelGGL(order_start_kernel, dim3(1), dim3(kWave), 0, stream, counts);
        hipLaunchKernelGGL(order_place_kernel, dim3(nb), dim3(256), 0, stream, p.off, p.n_scenarios, counts,
                           (int32_t*)p.order_ws + kOrderBuckets);
        const hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return e0;
    }
    const hipError_t e = launch_parts(p.n_scenarios, w * kWave, [&](dim3 grid, int64_t first) {
        ProjectParams q = p;
        q.first_block = first;
        hipLaunchKernelGGL(kern, grid, dim3(w * kWave), lds, stream, q);
    });
    if (e != hipSuccess || !p.rows) return e;
    const int64_t blocks = p.n_scenarios * ((p.H + kRowsThreads - 1) / kRowsThreads);
    const auto rows = p.nf == 4 ? expand_rows_kernel<4> : expand_rows_kernel<3>;
    return launch_parts(blocks, kRowsThreads, [&](dim3 grid, int64_t first) {
        ProjectParams q = p;
        q.first_block = first;
        hipLaunchKernelGGL(rows, grid, dim3(kRowsThreads), 0, stream, q);
    });
}

}  // namespace tl
