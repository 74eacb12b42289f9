// Which t_max candidates the recurrence is run for.
//
// F(s, k, d; t_max) of Eq. 3 is a minimum over the terms that pass the filter t_intra <= t_max, so
// min_s F(s, 1, N*M; t_max) never grows with t_max: over the ascending candidate list it is a
// staircase, and two evaluated candidates with the same value settle every candidate between
// them.  The staircases of model-like tables have few steps (99 over the 4096 candidates of the
// 64-layer expert workload on 8 x 8, 156 of 4096 and 223 of 7321 on the other two large ones), so the list is
// evaluated in rounds: evenly spaced knots first, then points inside the intervals whose ends differ,
// in the last round all of those.  What two knots cannot settle is evaluated; a table on which
// every candidate has a value of its own is evaluated whole, in the last round.
//
// The winner of Eq. 4 is always an evaluated candidate: T* = F + (B - 1) t_max takes the lowest
// t_max on ties, so within a step of the staircase the first candidate wins, and a candidate whose
// predecessor has another value is never strictly inside an interval with equal ends.
#include "internal.hpp"

namespace alpa {

constexpr int RF_THREADS = 1024;
constexpr int RF_WAVES = RF_THREADS / WAVE;

// Evenly spaced knot g of m over [0, n): both ends included.
__device__ __forceinline__ int even_knot(int g, int m, int n)
{
    return m <= 1 ? 0 : (int)(((long long)g * (n - 1)) / (m - 1));
}

// The candidates from the table's distinct values: all of them, or evenly spaced ones.  (by threads x of n)
__device__ __forceinline__ int pick_candidates(const PickQuery &pick, int32_t *cand, SolveState *state, int x, int n)
{
    const int m = (int)*pick.n_distinct;
    int C = (pick.n_quantiles == 0 || m <= pick.n_quantiles) ? m : pick.n_quantiles;
    if (C > pick.cap) C = pick.cap;
    const bool all = (C == m);
    for (int j = x; j < C; j += n)
        cand[j] = all ? pick.distinct[j] : pick.distinct[((long long)j * (m - 1)) / (pick.n_quantiles - 1)];
    if (x == 0) {
        state->n_cand = C;
        state->n_distinct = m;
    }
    return C;
}

__global__ void pick_candidates_kernel(PickQuery pick, int32_t *cand, SolveState *state)
{
    pick_candidates(pick, cand, state, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

__global__ void set_candidates_kernel(const uint32_t *__restrict__ n_unique_p, SolveState *state)
{
    state->n_cand = (int)*n_unique_p;
    state->n_distinct = (int)*n_unique_p;
}

// first index of the ascending candidates with a value of at least v (n: none)
__device__ __forceinline__ int first_at_least(const int32_t *__restrict__ cand, int n, int32_t v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cand[mid] >= v) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// first index in [lo, hi) with B * value >= U (hi: none)
__device__ __forceinline__ int first_product(const int32_t *__restrict__ cand, int lo, int hi, int64_t B, int64_t U)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (B * (int64_t)cand[mid] >= U) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// The range of candidates worth searching, and the first round's knots in it (one block).
//   * Below the smallest t_max with a plan (bounds) every candidate is infeasible.
//   * The first candidate j0 at or above it admits a plan of s stages, each at most that t_max, so
//     T*(j0) <= U = s t_feas + (B - 1) t_max(j0): with the early exit of Alg. 1, nothing from the first
//     candidate on with B t_max >= U is evaluated; where only the plan counts, a candidate
//     with (least unfiltered F) + (B - 1) t_max >= U cannot win against j0.
// (Where the bounds say nothing, t_feas is 0 and `stages` negative: everything is searched.)
// The list is sorted as unsigned, so values below zero (only a device-side list can hold them) come last;
// no entry passes them.
__global__ __launch_bounds__(RF_THREADS) void refine_begin_kernel(RefineQuery rq, int all, int first_round,
                                                                  PickQuery pick, int32_t *cand,
                                                                  SolveState *state,
                                                                  int32_t *__restrict__ knots,
                                                                  int32_t *__restrict__ list)
{
    __shared__ int sh_end, sh_first;
    constexpr int PLANS = BAND_THRESHOLDS + 2;
    __shared__ int32_t sh_sum[PLANS], sh_x[PLANS], sh_c[PLANS], sh_lo[PLANS];
    int C;
    if (pick.distinct) {
        C = pick_candidates(pick, cand, state, threadIdx.x, RF_THREADS);
        __syncthreads();
    } else {
        C = state->n_cand;
    }
    const int64_t t_feas = rq.bounds[rq.Smax + 1], stages = rq.bounds[rq.Smax + 2];
    const int32_t least_of_all = rq.bounds[0], flat = rq.bounds[rq.Smax + 3];
    int lo = 0, hi = C;                                // first index with a negative value
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cand[mid] < 0) hi = mid; else lo = mid + 1;
    }
    const int n = lo;
    lo = 0; hi = n;                                    // first index with a plan
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cand[mid] >= t_feas) hi = mid; else lo = mid + 1;
    }
    int j0 = t_feas >= DEV_INF ? n : lo;
    if (threadIdx.x == 0) {
        sh_end = (rq.prune || rq.plan_only) ? min(n, j0 + 1) : n;
        sh_first = rq.plan_only && rq.thr ? n : j0;
    }
    __syncthreads();
    if ((rq.prune || rq.plan_only) && rq.thr && j0 < n) {
        // Plans are known (of sum s and largest stage m: T* of the first candidate c that is not below m is at
        // most s + (B - 1) c), and for every candidate a lower bound on F.  Where the bounds come from the recurrence itself, so
        // are one of `stages` stages up to t_feas, and the least of all, whose stages are at most their sum.
        for (int t = threadIdx.x; t < PLANS; t += RF_THREADS) {
            const int j = min(t, BAND_THRESHOLDS - 1);
            int32_t sum = rq.thr[BAND_THRESHOLDS + 1 + 2 * j], largest = rq.thr[BAND_THRESHOLDS + 2 + 2 * j];
            if (t >= BAND_THRESHOLDS) {
                const bool feas = t == BAND_THRESHOLDS;
                sum = stages < 0 ? DEV_INF : feas ? (int32_t)(stages * t_feas) : least_of_all;
                largest = feas ? (int32_t)t_feas : least_of_all;
            }
            const int32_t above = band_threshold(rq.max_finite, j + 1 < BAND_THRESHOLDS ? j + 1 : j);
            const int x = first_at_least(cand, n, largest);
            sh_sum[t] = x < n ? sum : DEV_INF;
            sh_x[t] = min(x, n - 1);
            sh_c[t] = cand[min(x, n - 1)];
            // candidates that take threshold t: from sh_lo[t] on, up to the threshold
            sh_lo[t] = max(j0, j + 1 < BAND_THRESHOLDS ? first_at_least(cand, n, above + 1) : 0);
        }
        __syncthreads();
        const int lane = threadIdx.x & (WAVE - 1);
        for (int b = threadIdx.x >> 6; b < rq.n_B; b += RF_WAVES) {        // a wave per B value
            const int64_t B = rq.B_vals ? rq.B_vals[b] : rq.B;
            int64_t U = INF_I64;
            for (int t = lane; t < PLANS; t += WAVE)
                if (sh_sum[t] < DEV_INF) U = min64(U, sh_sum[t] + (B - 1) * (int64_t)sh_c[t]);
            U = wave_min_i64(U);
            int64_t lowest = (int64_t)n << 32;         // the lowest candidate known to reach U: its number, and its value
            for (int t = lane; t < PLANS; t += WAVE)
                if (sh_sum[t] < DEV_INF && sh_sum[t] + (B - 1) * (int64_t)sh_c[t] == U)
                    lowest = min64(lowest, (int64_t)sh_x[t] << 32 | sh_c[t]);
            lowest = wave_min_i64(lowest);
            const int at = hi32(lowest);
            // with the early exit nothing behind the first B t_max >= U is looked at; where only the plan counts, nothing that
            // cannot get below U (nor reach it before `at`).  What is left out must not set the early exit off either: at
            // candidates in front of `at` it cannot, as their t_max is below that plan's largest stage and B t_max below U;
            // but `at` itself may be far above the plan, so in front of it only what cannot get down to B t_max(at) goes
            int first = n, end = j0 + 1;
            if (U == INF_I64) {
                first = j0;
                end = n;
            } else {
                const int stop = rq.prune ? max(at + 1, first_product(cand, at + 1, n, B, U)) : n;
                end = stop;
                if (rq.plan_only) {
                    const int64_t in_front = rq.early_exit ? max(B * (int64_t)lo32(lowest), U) : U;
                    end = min(at + 1, n);
                    for (int t = lane; t < BAND_THRESHOLDS; t += WAVE) {
                        const int lo_t = sh_lo[t], hi_t = min(stop, t == 0 ? n : sh_lo[t - 1]);
                        const int64_t least = max(rq.thr[t], least_of_all), most = lo_t < at ? in_front : U;
                        if (lo_t >= hi_t || least >= DEV_INF || least + (B - 1) * (int64_t)cand[lo_t] > most) continue;
                        first = min(first, lo_t);
                        int x = lo_t, z = hi_t;        // first index that cannot get to `most`
                        while (x < z) {
                            const int mid = (x + z) >> 1;
                            if (least + (B - 1) * (int64_t)cand[mid] > most) z = mid; else x = mid + 1;
                        }
                        end = max(end, x);
                    }
                    first = min(first, at);
                }
            }
            first = wave_min_i32(first);
            end = -wave_min_i32(-end);
            if (lane == 0) {
                atomicMin(&sh_first, first);
                atomicMax(&sh_end, end);
            }
        }
        __syncthreads();
        j0 = max(j0, min(sh_first, sh_end - 1));
    } else if ((rq.prune || rq.plan_only) && j0 < n) {
        for (int b = threadIdx.x; b < rq.n_B; b += RF_THREADS) {
            const int64_t B = rq.B_vals ? rq.B_vals[b] : rq.B;
            const int64_t U = stages < 0 ? INF_I64 : stages * t_feas + (B - 1) * (int64_t)cand[j0];
            const int64_t least = rq.bounds[0];
            int x = j0 + 1, z = n;                     // first index in [x, z) that need not be looked at
            while (x < z) {
                const int mid = (x + z) >> 1;
                const int64_t c = cand[mid];
                if ((rq.prune && B * c >= U) || (rq.plan_only && least + (B - 1) * c >= U)) z = mid;
                else x = mid + 1;
            }
            atomicMax(&sh_end, x);
        }
        __syncthreads();
    }
    const int end = sh_end;
    // knots: evenly up to where the table says that F hardly changes any more, and the last candidate; where that is a guess,
    // a quarter of them evenly behind it
    lo = j0; hi = max(j0, end - 1);
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cand[mid] >= flat) hi = mid; else lo = mid + 1;
    }
    if (rq.heads && end - j0 > all) {
        // Candidates without a graph cost a workgroup each: where they are many, as many knots as without graphs
        __shared__ int sh_bare;
        __syncthreads();
        if (threadIdx.x == 0) sh_bare = 0;
        __syncthreads();
        for (int t = threadIdx.x; t < BAND_THRESHOLDS; t += RF_THREADS)
            if (rq.heads[t].n_stages < 0) {
                const int from = t + 1 < BAND_THRESHOLDS ? first_at_least(cand, n, band_threshold(rq.max_finite, t + 1) + 1) : 0;
                const int to = t == 0 ? n : first_at_least(cand, n, band_threshold(rq.max_finite, t) + 1);
                const int bare = min(to, end) - max(from, j0);
                if (bare > 0) atomicAdd(&sh_bare, bare);
            }
        __syncthreads();
        if (sh_bare > 512) first_round = min(first_round, 256);
    }
    const int span = lo + 1 - j0, rest = min(end - 1 - lo, stages == -1 ? 1 : first_round / 4);
    const bool whole = end - j0 <= all;
    const int m = whole ? end - j0 : min(first_round, span + rest);
    for (int j = threadIdx.x; j < m; j += RF_THREADS) {
        const int k = whole ? j0 + j : j < m - rest ? j0 + even_knot(j, m - rest, span) : lo + even_knot(j - (m - rest) + 1, rest + 1, end - lo);
        list[j] = k;
        if (j < REFINE_MAX_KNOTS) knots[j] = k;
    }
    // nothing outside [j0, end) is evaluated, read, or to be taken for a winner: in front of it nothing is feasible (or
    // gets to what a plan is known for), and behind it a lower candidate has the lowest possible T (with the early
    // exit they lie behind it)
    if (threadIdx.x == 0) {
        state->n_first = j0;
        state->n_range = end;
        state->n_list = m;
        state->n_knots = min(m, REFINE_MAX_KNOTS);
        state->clock[1] = wall_clock64();
        state->n_todo = 0;
        state->todo_ticket = 0;
        for (int x = 0; x < 4; ++x) state->thin[x] = 0;
    }
}

// Exclusive prefix sum of one value per thread over the block, and the block's total.
__device__ __forceinline__ int block_scan(int v, int *sh, int &total)
{
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const int o = __shfl_up(x, off, WAVE);
        if (lane >= off) x += o;
    }
    __syncthreads();                                   // sh may still be read from the last call
    if (lane == WAVE - 1) sh[w] = x;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < RF_WAVES; ++k) {
        const int t = sh[k];
        base += k < w ? t : 0;
        total += t;
    }
    return base + x - v;
}

// One step between two rounds (one block).  Reads F at the knots, decides which intervals between
// neighbouring knots still need points, and writes the next round's list; `last`: that is every
// point of those intervals, and the points of the others get their value here.
//
//   prune      the early exit of Alg. 1: nothing from the first index on at which
//              the knots alone show B * t_max >= best so far is needed.
//   plan_only  no per-candidate results are asked for: an interval is needed only if one of its points
//              could still beat the best knot at or below it, i.e. its lower bound
//              F(right end) + (B - 1) t_max(first point) is below that knot's T* for one of the B
//              values.  The points of the others take the left end's F, an upper bound that
//              leaves every prefix minimum (and with it the early exit) as it is.
// Otherwise a step takes at most `budget` points, dealt to the intervals in proportion to their
// lengths.
__global__ __launch_bounds__(RF_THREADS) void refine_kernel(
    RefineQuery rq, const int32_t *__restrict__ cand, int32_t *__restrict__ Fmin, SolveState *state,
    int last, int budget, const int32_t *__restrict__ knots, int32_t *__restrict__ knots_out, int32_t *__restrict__ list)
{
    __shared__ int32_t kx[REFINE_MAX_KNOTS];           // knot positions
    __shared__ int32_t kf[REFINE_MAX_KNOTS];           // F there
    __shared__ int32_t kn[REFINE_MAX_KNOTS];           // points wanted right of the knot
    __shared__ int sh[RF_WAVES];
    __shared__ int sh_range;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid >> 6;
    const int prune = rq.prune, plan_only = rq.plan_only;
    const int m = state->n_knots;
    int range = state->n_range;
    for (int i = tid; i < m; i += RF_THREADS) {
        const int x = knots[i];
        kx[i] = x;
        kf[i] = Fmin[x];
    }
    if (tid == 0) sh_range = range;
    __syncthreads();
    for (int i = tid; i < m; i += RF_THREADS)
        kn[i] = (!plan_only && i + 1 < m && kf[i] != kf[i + 1]) ? kx[i + 1] - kx[i] - 1 : 0;
    __syncthreads();
    if (prune || plan_only) {
        // a wave per B value (the waves without one sit this out)
        for (int b = w; b < rq.n_B; b += RF_WAVES) {
            const int64_t B = rq.B_vals ? rq.B_vals[b] : rq.B;
            int64_t carry = INF_I64;
            for (int i0 = 0; i0 < m; i0 += WAVE) {
                const int i = i0 + lane;
                int64_t t = INF_I64;
                int64_t c = 0;
                if (i < m) {
                    c = cand[kx[i]];
                    if (kf[i] < DEV_INF) t = (int64_t)kf[i] + (B - 1) * c;
                }
                const int64_t incl = min64(wave_prefix_min_i64(t, lane), carry);
                if (plan_only && i + 1 < m && kf[i] != kf[i + 1] && kx[i + 1] - kx[i] > 1) {
                    const int64_t lb = (int64_t)kf[i + 1] + (B - 1) * (int64_t)cand[kx[i] + 1];
                    if (lb < incl) kn[i] = kx[i + 1] - kx[i] - 1;      // same value from any wave
                }
                if (prune) {
                    // first knot at which the rule fires on the knots before it
                    const int lo = __shfl_up(lo32(incl), 1, WAVE), hi = __shfl_up(hi32(incl), 1, WAVE);
                    const int64_t excl = lane == 0 ? carry : i64_from(lo, hi);
                    const uint64_t hit = __ballot(i < m && i > 0 && excl != INF_I64 && B * c >= excl);
                    if (hit) {
                        const int at = __ffsll((unsigned long long)hit) - 1;
                        const int64_t e = i64_from(__shfl(lo32(excl), at, WAVE), __shfl(hi32(excl), at, WAVE));
                        int a = kx[i0 + at - 1] + 1, z = kx[i0 + at];   // it fires in [a, z]
                        while (a < z) {
                            const int mid = (a + z) >> 1;
                            if (B * (int64_t)cand[mid] >= e) z = mid; else a = mid + 1;
                        }
                        sh_range = a;                  // one B value with the early exit
                        break;
                    }
                }
                carry = i64_from(__shfl(lo32(incl), WAVE - 1, WAVE), __shfl(hi32(incl), WAVE - 1, WAVE));
            }
        }
        __syncthreads();
        range = min(range, sh_range);
    }
    // how many points each interval gets, and where they go
    int mine = 0;
    for (int i = tid; i < m; i += RF_THREADS) {
        const int g = max(0, min(kn[i], range - kx[i] - 1));
        kn[i] = g;
        mine += g;
    }
    int total;
    (void)block_scan(mine, sh, total);
    const bool everything = last || total <= budget;
    int list_base = 0, len_base = 0;
    for (int i0 = 0; i0 < m; i0 += RF_THREADS) {
        const int i = i0 + tid;
        const int g = i < m ? kn[i] : 0;
        int t0, t1;
        const int before = len_base + block_scan(g, sh, t0);
        int take = g;
        if (!everything)                               // (all intervals together: `budget` points)
            take = (int)(((long long)(before + g) * budget) / total) -
                   (int)(((long long)before * budget) / total);
        const int at = list_base + block_scan(take, sh, t1);
        if (i < m) {
            // a short share is written here; longer ones by whole waves below
            kn[i] = take;
            if (!last) knots_out[i + at] = kx[i];
            for (int u = 0; u < take && take <= 4; ++u) {
                const int j = everything ? kx[i] + 1 + u
                                         : kx[i] + (int)(((long long)(g + 1) * (u + 1)) / (take + 1));
                list[at + u] = j;
                if (!last) knots_out[i + at + 1 + u] = j;
            }
        }
        // (a wave's lanes hold 64 neighbouring intervals; its long ones one after the other)
        for (uint64_t todo = __ballot(take > 4); todo; todo &= todo - 1) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const int tk = __shfl(take, l, WAVE), ap = __shfl(at, l, WAVE), gp = __shfl(g, l, WAVE);
            const int s = i0 + w * WAVE + l, x = kx[s];
            for (int u = lane; u < tk; u += WAVE) {
                const int j = everything ? x + 1 + u : x + (int)(((long long)(gp + 1) * (u + 1)) / (tk + 1));
                list[ap + u] = j;
                if (!last) knots_out[s + ap + 1 + u] = j;
            }
        }
        len_base += t0;
        list_base += t1;
    }
    if (last) {
        // every point that no round evaluates: its interval's ends agree, or it cannot matter
        __syncthreads();
        for (int i = w; i + 1 < m; i += RF_WAVES) {
            if (kn[i] != 0) continue;
            const int end = min(kx[i + 1], range);
            for (int j = kx[i] + 1 + lane; j < end; j += WAVE) Fmin[j] = kf[i];
        }
    }
    if (tid == 0) {
        state->n_range = range;
        state->n_list = list_base;
        state->n_knots = last ? m : m + list_base;
        state->ticket = 0;
        state->n_todo = 0;
        state->todo_ticket = 0;
        for (int x = 0; x < 4; ++x) state->thin[x] = 0;
    }
}

// Up to PICK_HERE candidates are picked by the block that begins the first round (a launch of its own is 4 us of the stream's time; eight
// turns of the block's threads are 3).
constexpr int PICK_HERE = 8192;

hipError_t launch_pick_candidates(hipStream_t st, PickQuery &pick, int bound, int32_t *cand, SolveState *state)
{
    if (bound <= PICK_HERE) return hipSuccess;
    const int grid = std::max(1, std::min((bound + 255) / 256, 1024));
    hipLaunchKernelGGL(pick_candidates_kernel, dim3(grid), dim3(256), 0, st, pick, cand, state);
    pick.distinct = nullptr;
    return hipGetLastError();
}

hipError_t launch_set_candidates(hipStream_t st, const uint32_t *n_unique, SolveState *state)
{
    hipLaunchKernelGGL(set_candidates_kernel, dim3(1), dim3(1), 0, st, n_unique, state);
    return hipGetLastError();
}

hipError_t launch_refine_begin(hipStream_t st, const RefineQuery &rq, const PickQuery &pick, int32_t *cand, SolveState *state,
                               const RefineBuffers &rb)
{
    hipLaunchKernelGGL(refine_begin_kernel, dim3(1), dim3(RF_THREADS), 0, st, rq, rb.all, rb.first_round, pick, cand,
                       state, rb.knots[0], rb.list);
    return hipGetLastError();
}

hipError_t launch_refine(hipStream_t st, const RefineQuery &rq, const int32_t *cand, int32_t *Fmin,
                         SolveState *state, int round, int last, const RefineBuffers &rb)
{
    hipLaunchKernelGGL(refine_kernel, dim3(1), dim3(RF_THREADS), 0, st, rq, cand, Fmin, state, last, rb.budget,
                       rb.knots[(round - 1) & 1], rb.knots[round & 1], rb.list);
    return hipGetLastError();
}

}  // namespace alpa
