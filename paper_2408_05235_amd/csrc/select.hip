// Stage 3: the throttling controller (Sec. 4.5) with the TBT and E2E checks of
// Sec. 4.3.2 (checks 2 and 3, Eq. 3-4).
//
// One 256-thread workgroup per scenario; its four wavefronts take the
// candidate frequencies in rounds of four, lowest first, and the first round
// with a feasible frequency ends the search.  For one frequency a wave walks
// the projected iterations 256 at a time, four consecutive ones per lane:
// per-iteration time in integer ns, the lane's running sum plus an exclusive
// wave scan of lane totals and the carry gives Eq. 3's cumulative time
// T_R[j+1], which is compared with the deadline of requests ending at j.  The
// walk stops at the first violated deadline.
//
// The admission decision of Sec. 4.3.2 and the steps of the paper's binary
// search over frequencies use the same arithmetic at one frequency per
// scenario.
#include "device_util.h"
#include "tl_internal.h"

namespace tl {
namespace {

constexpr uint64_t kNoDeadline = ~0ull;
constexpr uint64_t kSat = 1ull << 40;

// T'_j = 1 / T_j in whole ns, rounded up; IEEE fp64 division
__device__ __forceinline__ uint64_t latency_ns(float ips) {
    if (!(ips > 0.0f)) return kSat;
    const double q = 1e9 / (double)ips;
    if (!(q < 1099511627776.0)) return kSat;
    return (uint64_t)ceil(q);
}

constexpr int kWavesPerBlock = 4;
constexpr int kPerLane = 4;                   // consecutive iterations per lane
constexpr int kStep = kWave * kPerLane;       // iterations per wavefront step

// Eq. 3-4 for one frequency, by one wavefront: per-iteration times of `ips`
// over the n projected iterations, T_R[j+1] < dl[j] for every deadline and
// T_R[n] <= budget.  A lane takes four consecutive iterations: their running
// sum, then one wave scan of the lane totals per 256 iterations.  Stops at
// the first missed deadline.  Every lane returns the same value.
__device__ __forceinline__ bool feasible_wave(const float* ips, const uint64_t* dl, int32_t n, uint64_t budget) {
    const int lane = lane_id();
    uint64_t carry = 0;
    for (int32_t j0 = 0; j0 < n; j0 += kStep) {
        const int32_t jb = j0 + kPerLane * lane;
        uint64_t p[kPerLane];
        uint64_t run = 0;
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            run += (jb + k < n) ? latency_ns(ips[jb + k]) : 0ull;
            p[k] = run;
        }
        const uint64_t before = wave_incl_scan_u64(run) - run + carry;   // T_R[jb]
        bool bad = false;
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            if (jb + k < n) {
                const uint64_t d = dl[jb + k];
                bad |= d != kNoDeadline && !(before + p[k] < d);
            }
        }
        carry = lane63_u64(before + run);
        if (__ballot(bad)) return false;
    }
    return carry <= budget;
}

// The lowest feasible frequency of one scenario.  The four wavefronts of the
// workgroup take frequencies in rounds of four, lowest first; the first
// round with a feasible frequency ends the search (no higher frequency can
// be the minimum).
__global__ __launch_bounds__(256) void select_kernel(SelectParams P) {
    __shared__ uint32_t round_ok;
    const int64_t s = P.first_block + blockIdx.x;
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int32_t F = P.F, H = P.H;
    const uint32_t fl = P.proj_flags ? P.proj_flags[s] : 0u;
    if (fl & (TL_FLAG_OVERFLOW | TL_FLAG_LOST)) {
        if (threadIdx.x == 0) {
            P.freq_idx[s] = F - 1;
            P.status[s] = (fl & TL_FLAG_OVERFLOW) ? TL_STATUS_INVALID : TL_STATUS_LOST;
        }
        return;
    }
    const int32_t n = min(max(P.n_iters[s], 0), H);
    if (n == 0) {
        if (threadIdx.x == 0) {
            P.freq_idx[s] = 0;
            P.status[s] = TL_STATUS_OK;
        }
        return;
    }
    if (threadIdx.x == 0) round_ok = 0;
    __syncthreads();
    const uint64_t slo = P.tbt_slo_ns[s];
    const uint64_t budget = (slo > ~0ull / (uint64_t)n) ? ~0ull : slo * (uint64_t)n;
    const uint64_t* dl = P.deadline_at + s * H;
    int32_t best = -1;
    for (int32_t f0 = 0; f0 < F; f0 += kWavesPerBlock) {
        const int32_t f = f0 + wave;
        const bool ok = f < F && feasible_wave(P.ips + ((int64_t)s * F + f) * H, dl, n, budget);
        if (ok && lane == 0) atomicOr(&round_ok, 1u << wave);
        __syncthreads();
        const uint32_t m = round_ok;
        // every thread has read this round's mask before the next round writes
        __syncthreads();
        if (m) {
            best = f0 + __ffs(m) - 1;
            break;
        }
    }
    if (threadIdx.x == 0) {
        P.freq_idx[s] = best >= 0 ? best : F - 1;
        P.status[s] = best >= 0 ? TL_STATUS_OK : TL_STATUS_INFEASIBLE;
    }
}

// Eq. 3 at one frequency over iterations [r0, r1) of one scenario, by one
// wavefront, PER consecutive iterations a lane: with T_R[r0] = carry, whether some
// deadline of `dl` (T_R[j+1] < dl[j]) is missed on a lane (*miss), and whether
// T_R[own_at + 1] < d_own fails (*miss_own).  Returns T_R[r1].
template <int PER>
__device__ __forceinline__ uint64_t run_times(const float* ips, const uint64_t* dl, int32_t r0, int32_t r1,
                                              uint64_t carry, int32_t own_at, uint64_t d_own, bool* miss,
                                              bool* miss_own) {
    for (int32_t j0 = r0; j0 < r1; j0 += kWave * PER) {
        const int32_t jb = j0 + PER * lane_id();
        uint64_t t[PER], step = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            step += jb + k < r1 ? latency_ns(ips[jb + k]) : 0ull;
            t[k] = step;
        }
        const uint64_t before = wave_incl_scan_u64(step) - step + carry;   // T_R[jb]
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (jb + k < r1) {
                const uint64_t d = dl[jb + k];
                *miss |= d != kNoDeadline && !(before + t[k] < d);
                *miss_own |= jb + k == own_at && !(before + t[k] < d_own);
            }
        carry = lane63_u64(before + step);
    }
    return carry;
}

// Eq. 3-4 at one frequency for one scenario, by W wavefronts: with
// per-iteration times of `ips` over the n projected iterations, returns T_R[n]
// and whether some deadline of `dl` is missed; *miss_own tells whether
// T_R[own_at + 1] < d_own fails (own_at < 0: none).  Every thread returns the
// same values; all of them call it.
// W = 4, a workgroup: each wavefront takes a run of consecutive iterations, its
// run's total first, then, from the totals of the wavefronts before it, the times
// of its iterations.  (One wavefront stepping through the iterations 64 at a time
// was a chain of loads and scans: 13 us for 2048 iterations, however few the
// scenarios.)  W = 1: one wavefront on its own, four scenarios a workgroup.
constexpr int kTimeWaves = 4;
constexpr int kTimeThreads = kTimeWaves * kWave;

template <int W>
__device__ __forceinline__ uint64_t scenario_times(const float* ips, const uint64_t* dl, int32_t n, int32_t own_at,
                                                   uint64_t d_own, bool* miss, bool* miss_own) {
    bool m = false, mo = false;
    if (W == 1) {
        const uint64_t all = n <= kWave ? run_times<1>(ips, dl, 0, n, 0, own_at, d_own, &m, &mo)
                                        : run_times<kPerLane>(ips, dl, 0, n, 0, own_at, d_own, &m, &mo);
        *miss = __ballot(m) != 0;
        *miss_own = __ballot(mo) != 0;
        return all;
    }
    __shared__ uint64_t totals[kTimeWaves];
    __shared__ uint32_t missed[2];
    const int wave = threadIdx.x / kWave;
    const int32_t run = (n + kTimeWaves * kStep - 1) / (kTimeWaves * kStep) * kStep;
    const int32_t r0 = min(wave * run, n), r1 = min(r0 + run, n);
    if (threadIdx.x == 0) missed[0] = missed[1] = 0;
    uint64_t sum = 0;
    for (int32_t j0 = r0; j0 < r1; j0 += kStep) {
        const int32_t jb = j0 + kPerLane * lane_id();
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) sum += jb + k < r1 ? latency_ns(ips[jb + k]) : 0ull;
    }
    sum = wave_sum_u64(sum);
    if (lane_id() == 0) totals[wave] = sum;
    __syncthreads();
    uint64_t carry = 0, all = 0;   // T_R[r0] and T_R[n]
#pragma unroll
    for (int w = 0; w < kTimeWaves; ++w) {
        if (w < wave) carry += totals[w];
        all += totals[w];
    }
    run_times<kPerLane>(ips, dl, r0, r1, carry, own_at, d_own, &m, &mo);
    if (m) missed[0] = 1;
    if (mo) missed[1] = 1;
    __syncthreads();
    *miss = missed[0] != 0;
    *miss_own = missed[1] != 0;
    return all;
}

// The scenario of this workgroup (W = 4) or wavefront (W = 1).
template <int W>
__device__ __forceinline__ int64_t time_scenario(int64_t first_block) {
    const int64_t block = first_block + blockIdx.x;
    return W == 1 ? block * kTimeWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) : block;
}
template <int W>
__device__ __forceinline__ int time_thread() {
    return W == 1 ? lane_id() : (int)threadIdx.x;
}

// Wavefronts per scenario of the checks at one frequency: four where they
// shorten a chain of steps and the device has room for them.  Measured (us, a
// search over 17 frequencies by table, five checks; one / four wavefronts):
// 2048 scenarios x 256 iterations 42 / 46, x 1024 94 / 91, x 2048 156 / 145;
// 4096 x 64 41 / 63, x 1024 134 / 149, x 4096 517 / 555; 65536 x 16 226 / 721; 64
// x 256 41 / 41, x 4096 117 / 65.
int time_waves(int64_t S, int32_t H) { return S > 2048 || H <= kStep ? 1 : kTimeWaves; }

__device__ __forceinline__ bool within_tbt(uint64_t t_r_n, uint64_t slo, int32_t n) {
    const uint64_t budget = n == 0 ? ~0ull : (slo > ~0ull / (uint64_t)n) ? ~0ull : slo * (uint64_t)n;
    return t_r_n <= budget;
}

// Admission decision (Sec. 4.3.2 checks 1-3) of one new query per scenario
// from the projection with it and M at the maximum frequency: one workgroup
// or wavefront per scenario; the deadline of the query itself (ending at cand_len, when
// inside the horizon) is checked apart from the scheduled requests'
// deadlines in deadline_at.
template <int W>
__global__ __launch_bounds__(kTimeThreads) void admit_kernel(AdmitParams P) {
    const int64_t s = time_scenario<W>(P.first_block);
    if (s >= P.S) return;
    const int32_t H = P.H;
    const uint32_t fl = P.proj_flags[s];
    uint32_t dec;
    if (fl & (TL_FLAG_OVERFLOW | TL_FLAG_BAD_CANDIDATE)) {
        dec = TL_ADMIT_INVALID;
    } else if (fl & TL_FLAG_OVERCOMMIT) {
        // the requests running now (the query among them) exceed the KV
        // capacity at some iteration or the batch cap: every value of the
        // projected KV vector is within the capacity otherwise, since queued
        // requests are only admitted where they fit
        dec = TL_ADMIT_QUEUE_CAPACITY;
    } else {
        const int32_t n = min(max(P.n_iters[s], 0), H);
        const int32_t L = P.cand_len[s];
        const uint64_t d_own = P.cand_deadline ? P.cand_deadline[s] : kNoDeadline;
        const int32_t own_at = (d_own != kNoDeadline && L <= H) ? L - 1 : -1;   // T_R[L] = T_R[own_at + 1]
        bool miss, miss_own;
        const uint64_t t_r =
            scenario_times<W>(P.ips + s * H, P.deadline_at + s * H, n, own_at, d_own, &miss, &miss_own);
        if (!within_tbt(t_r, P.tbt_slo_ns[s], n)) dec = TL_ADMIT_QUEUE_TBT;
        else if (miss) dec = TL_ADMIT_QUEUE_E2E;
        else if (miss_own) dec = TL_ADMIT_LOST;
        else dec = TL_ADMIT_OK;
    }
    if (time_thread<W>() == 0) P.decision[s] = dec;
}

// Binary search over the candidate frequencies (Sec. 4.5), one step per
// launch for every scenario.  State per scenario: lo, hi (the search
// interval) and probe (the frequency index M was evaluated at, -1 = none).
// Step: feasible at the probe -> hi = probe, else lo = probe + 1; then the
// next probe is the midpoint while lo < hi.  The last step (final = true)
// checks lo itself and writes the result.  Scenarios flagged overflow / lost
// are settled by the first step (mode init) without probes.
// One workgroup or wavefront per scenario; the init, without times to add up,
// one thread.
__global__ __launch_bounds__(kTimeThreads) void search_init_kernel(SearchParams P) {
    const int64_t s = (int64_t)blockIdx.x * kTimeThreads + threadIdx.x;
    if (s >= P.S) return;
    const int32_t F = P.F;
    const uint32_t fl = P.proj_flags ? P.proj_flags[s] : 0u;
    const bool settled = (fl & (TL_FLAG_OVERFLOW | TL_FLAG_LOST)) != 0;
    P.work[s] = settled ? -1 : 0;
    P.work[P.S + s] = settled ? -1 : F - 1;
    P.work[2 * P.S + s] = (settled || F == 1) ? -1 : (F - 1) / 2;
    if (settled) {
        P.freq_idx[s] = F - 1;
        P.status[s] = (fl & TL_FLAG_OVERFLOW) ? TL_STATUS_INVALID : TL_STATUS_LOST;
    }
}

template <int W>
__global__ __launch_bounds__(kTimeThreads) void search_kernel(SearchParams P, int mode) {
    const int64_t s = time_scenario<W>(P.first_block);
    if (s >= P.S) return;
    int32_t* lo = P.work;
    int32_t* hi = P.work + P.S;
    int32_t* probe = P.work + 2 * P.S;
    const int32_t F = P.F, H = P.H;
    const int32_t p = probe[s];
    if (p < 0) return;
    const int32_t n = min(max(P.n_iters[s], 0), H);
    bool miss, miss_own;
    const uint64_t t_r =
        scenario_times<W>(P.ips + s * H, P.deadline_at + s * H, n, -1, kNoDeadline, &miss, &miss_own);
    const bool ok = !miss && within_tbt(t_r, P.tbt_slo_ns[s], n);
    if (time_thread<W>() != 0) return;
    if (mode == 2) {   // final check of lo
        P.freq_idx[s] = ok ? p : F - 1;
        P.status[s] = ok ? TL_STATUS_OK : TL_STATUS_INFEASIBLE;
        probe[s] = -1;
        return;
    }
    int32_t l = lo[s], h = hi[s];
    if (ok) h = p;
    else l = p + 1;
    lo[s] = l;
    hi[s] = h;
    probe[s] = l < h ? l + (h - l) / 2 : -1;
}

// Before the final check, lo == hi for every unsettled scenario.  hi only
// moves to a probe found feasible, and no probe is ever F-1 (the midpoint of
// lo < hi lies below hi), so hi < F-1 means lo was probed and found
// feasible: the scenario is settled here with lo (OK), as the final check of
// lo would settle it.  The others (hi still F-1) probe lo.
__global__ __launch_bounds__(256) void search_final_probe_kernel(SearchParams P) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= P.S) return;
    const int32_t l = P.work[s], h = P.work[P.S + s];
    const bool known = l >= 0 && l == h && h < P.F - 1;
    if (known) {
        P.freq_idx[s] = l;
        P.status[s] = TL_STATUS_OK;
    }
    P.work[2 * P.S + s] = known ? -1 : l;   // -1 stays -1 (settled)
}

}  // namespace

hipError_t launch_admit(const AdmitParams& p, hipStream_t stream) {
    const bool one = time_waves(p.S, p.H) == 1;
    const auto kern = one ? admit_kernel<1> : admit_kernel<kTimeWaves>;
    return launch_parts(one ? (p.S + kTimeWaves - 1) / kTimeWaves : p.S, kTimeThreads, [&](dim3 grid, int64_t first) {
        AdmitParams q = p;
        q.first_block = first;
        hipLaunchKernelGGL(kern, grid, dim3(kTimeThreads), 0, stream, q);
    });
}

hipError_t launch_search_step(const SearchParams& p, int mode, hipStream_t stream) {
    if (p.S == 0) return hipSuccess;
    if (mode == 3) {
        hipLaunchKernelGGL(search_final_probe_kernel, dim3((unsigned)((p.S + 255) / 256)), dim3(256), 0, stream, p);
    } else if (mode == 0) {
        hipLaunchKernelGGL(search_init_kernel, dim3((unsigned)((p.S + kTimeThreads - 1) / kTimeThreads)),
                           dim3(kTimeThreads), 0, stream, p);
    } else {
        const bool one = time_waves(p.S, p.H) == 1;
        const auto kern = one ? search_kernel<1> : search_kernel<kTimeWaves>;
        const int64_t blocks = one ? (p.S + kTimeWaves - 1) / kTimeWaves : p.S;
        return launch_parts(blocks, kTimeThreads, [&](dim3 grid, int64_t first) {
            SearchParams q = p;
            q.first_block = first;
            hipLaunchKernelGGL(kern, grid, dim3(kTimeThreads), 0, stream, q, mode);
        });
    }
    return hipGetLastError();
}

hipError_t launch_select(const SelectParams& p, hipStream_t stream) {
    return launch_parts(p.S, kWavesPerBlock * kWave, [&](dim3 grid, int64_t first) {
        SelectParams q = p;
        q.first_block = first;
        hipLaunchKernelGGL(select_kernel, grid, dim3(kWavesPerBlock * kWave), 0, stream, q);
    });
}

}  // namespace tl
