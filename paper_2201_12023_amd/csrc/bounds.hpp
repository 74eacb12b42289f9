// What the thresholds say about a table as a whole (kernels_band.hip, kernels_sparse.hip; gfx950 only).
#pragma once
#include "internal.hpp"

namespace alpa {

// the least sum of the thresholds' plans
__device__ __forceinline__ int32_t band_best_plan(const int32_t *plans)
{
    int32_t best = DEV_INF;
    for (int j = threadIdx.x & (WAVE - 1); j < BAND_THRESHOLDS; j += WAVE) best = min(best, plans[2 * j]);
    return wave_min_i32(best);
}

// Do the thresholds say little?  Then their best plan is far above P(K, D) without a filter (latencies without any order).
__device__ __forceinline__ bool band_bounds_poor(const int32_t *totals, int32_t best)
{
    return totals[0] < DEV_INF && best - totals[0] > (totals[0] >> 2);
}

// A plan of threshold j that is a real one, walked from its last stage on: how many stages lie behind each is known now, so every
// step takes the term that is least with the t_intra it really has in front of P.  plan[0] = the sum, plan[1] = the largest; as they
// were if it ends nowhere.
__device__ __forceinline__ void band_real_plan(const int32_t *__restrict__ table, const BandShapes &bs, const Problem &p, int32_t c,
                                               const int32_t *__restrict__ front, int RS, int32_t *plan)
{
    __shared__ unsigned long long sh_term[2];
    const int K = p.K, tid = threadIdx.x, nt = blockDim.x;
    if (tid < 2) sh_term[tid] = ~0ull;
    __syncthreads();
    int k = K, d = p.D;
    int32_t sum = 0, largest = 0;
    for (int n = 0; k > 0; ++n) {                  // (uniform: every thread walks the same plan)
        unsigned long long at = ~0ull;             // sum of the term and P, first layer, shape
        for (int b = tid >> 4; b < k; b += nt / 16)
            for (int q = tid & 15; q < bs.S; q += 16) {
                const int left = d - bs.sizes[q];  // P(b, left); no layer in front takes no device
                if (left < 0) continue;
                const int32_t f = b > 0 ? front[b * RS + p.D - left - 1] : left == 0 ? 0 : DEV_INF;
                const int32_t t = band_smallest(table + ((size_t)n * K * K + b * K + k - 1) * bs.S_table, bs, q);
                if (f < DEV_INF && t <= c) at = min(at, (unsigned long long)(t + f) << 32 | (unsigned)(b * 64 + q));
            }
        if (at != ~0ull) atomicMin(&sh_term[n & 1], at);
        __syncthreads();
        const unsigned long long x = sh_term[n & 1];
        if (x == ~0ull) return;
        const int b = (int)((uint32_t)x >> 6), q = (int)(x & 63);
        if (tid == 0) sh_term[~n & 1] = ~0ull;     // (last read a barrier ago)
        const int32_t t = band_smallest(table + ((size_t)n * K * K + b * K + k - 1) * bs.S_table, bs, q);
        k = b;
        d -= bs.sizes[q];
        sum += t;
        largest = max(largest, t);
        __syncthreads();
    }
    if (tid == 0) {
        plan[0] = sum;
        plan[1] = largest;
    }
}

// Bounds as launch_table_bounds writes them, from the thresholds: no plan of any number of stages is below P(K, D) without a filter,
// and the number of stages of a plan at the smallest t_max is not known.  From where on F hardly changes: the lowest threshold
// with that least sum, if the plan that reaches it is a real one (-1 for the stages).  Where it is not (a stage does not fit
// with many behind it, stages of equal layers, latencies without any order) it is the largest stage of the best plan (-2: a
// guess), and nowhere if that is far above.  If no threshold has a real plan, a workgroup for each looks for one, and
// the last to end writes the bounds: 48 layers on 32 x 8 with little memory have P 41184, plans of 41412 are found, the best of all is
// 41382 (the plan alone out of 300 candidates: 2050 us without a known plan, 606 with). (The thresholds' plans
// stay as they are until every workgroup has ended, as does `there`.)
__device__ __forceinline__ void band_bounds(const Problem &p, int32_t max_finite, const int32_t *__restrict__ table, const BandShapes &bs,
                                            const int32_t *__restrict__ fronts, int RS, const int32_t *__restrict__ totals, int32_t *plans,
                                            int32_t *__restrict__ bounds, int32_t *there, int j)
{
    __shared__ int32_t flat, own[2];
    __shared__ int last;
    const int tid = threadIdx.x;
    int32_t *const n_ended = plans + 2 * BAND_THRESHOLDS, *const real = n_ended + 1;
    int32_t best = band_best_plan(plans);
    const bool none = totals[0] < DEV_INF && best >= DEV_INF;
    if (none) {
        if (tid < 2) own[tid] = DEV_INF;
        __syncthreads();
        if (totals[j] < DEV_INF)
            band_real_plan(table, bs, p, band_threshold(max_finite, j), fronts + (size_t)j * p.K * RS, RS, own);
    }
    __syncthreads();
    if (tid == 0) {
        if (none) {
            __hip_atomic_store(&real[2 * j], own[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&real[2 * j + 1], own[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        last = __hip_atomic_fetch_add(n_ended, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    if (none) {
        for (int x = tid; x < 2 * BAND_THRESHOLDS; x += blockDim.x)
            plans[x] = __hip_atomic_load(&real[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        best = band_best_plan(plans);
    }
    const bool reached = totals[0] >= DEV_INF || plans[0] == totals[0], poor = band_bounds_poor(totals, best);
    if (tid == 0) flat = DEV_INF;
    __syncthreads();
    if (tid < BAND_THRESHOLDS) {
        if (reached && totals[tid] == totals[0]) atomicMin(&flat, band_threshold(max_finite, tid));
        if (!reached && !poor && plans[2 * tid] == best) atomicMin(&flat, plans[2 * tid + 1]);
    }
    __syncthreads();
    for (int s = tid; s <= p.Smax; s += blockDim.x) bounds[s] = totals[0];
    if (tid == 0) {
        bounds[p.Smax + 1] = totals[BAND_THRESHOLDS];
        bounds[p.Smax + 2] = reached ? -1 : -2;
        bounds[p.Smax + 3] = flat;
        *there = 1;
    }
}

}  // namespace alpa
