// Front costs: the least sum of stages that cover the first k layers on d devices, and what they say about a table.
//
//   P(k, d) = min over b < k and shapes of a devices of  least(b, k - 1, a) + P(b, d - a),   P(0, 0) = 0,
// where least(b, i, a) is the least latency of the stage of layers b .. i over the numbers of stages behind it, as far as it
// passes the filter.  Q(k, d) is the same from the back: the layers from k on, on d devices.  No plan is below P(K, D), and
// none that goes through the cell (k, d), with the layers from k on on d devices, is below P(k, D - d) + Q(k, d).
#include "internal.hpp"
#include "front.hpp"

#include <type_traits>

namespace alpa {

size_t front_least_ints(int K, int S) { return (size_t)K * K * front_padded(S); }
size_t front_table_ints(int K, int S) { return front_least_ints(K, S) / 4 + 2 * (size_t)front_units(K, S) * 65; }

FrontTable front_table(const int32_t *least, const int32_t *front, int K, int S, const int32_t *sizes, bool back)
{
    const int n = front_units(K, S);
    const int32_t *units = front + front_least_ints(K, S) / 4 + (back ? (size_t)n * 65 : 0);
    return FrontTable{units, units + (size_t)n * 64, least, (const uint8_t *)front, sizes, front_groups(S)};
}

// least[b][i][q] and run[b][i][q] (q padded to front_padded): the least latency over the numbers of stages behind, and with how
// many, itself included, the stage has it from one on.
__global__ __launch_bounds__(256) void front_least_kernel(const int32_t *__restrict__ table, int K, int Smax, BandShapes bs, int SP,
                                                          int32_t *__restrict__ least,
                                                          uint8_t *__restrict__ run)
{
    const int n = K * K * SP;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x) {
        const int ki = x / SP, q = x - ki * SP, k = ki / K, i = ki - k * K;
        int32_t m = INF_I32;
        int leading = 0;
        if (q < bs.S && i >= k) {
            const int32_t *t = table + (size_t)ki * bs.S_table;
            const size_t layer = (size_t)K * K * bs.S_table;
            for (int y = bs.first ? bs.first[q] : q; y >= 0; y = bs.first ? bs.next[y] : -1) {
                const int32_t first = t[y];
                leading = 0;
#pragma unroll 8
                for (int s = 0; s < Smax; ++s) {
                    const int32_t v = t[s * layer + y];
                    leading += v == first && leading == s;
                    m = min(m, v);
                }
            }
        }
        least[x] = min(m, DEV_INF);
        run[x] = (uint8_t)leading;
    }
}

// The units from `least`, a wave each; blockIdx.y: those of P, those of Q (the layers in reverse order)
__global__ __launch_bounds__(256) void front_units_kernel(const int32_t *__restrict__ least, int K, int S, int SP,
                                                          int32_t *__restrict__ units)
{
    const int lane = threadIdx.x & (WAVE - 1), NG = front_groups(S), n = front_units(K, S);
    const bool back = blockIdx.y == 1;
    units += back ? (size_t)n * 65 : 0;
    int32_t *const unit_min = units + (size_t)n * 64;
    for (int u = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6); u < n; u += gridDim.x * (blockDim.x / WAVE)) {
        const int g = u % NG, x = u / NG;
        int J = 0;                                 // the block: units_before(J) <= x
        while (front_units_before(J + 1) <= x) ++J;
        const int b = x - front_units_before(J), i = 8 * J + ((lane >> 2) & 7), q = 8 * g + 2 * (lane & 3) + (lane >> 5);
        int32_t t = DEV_INF;
        if (b <= i && i < K && q < S) t = back ? least[((size_t)(K - 1 - i) * K + K - 1 - b) * SP + q] : least[((size_t)b * K + i) * SP + q];
        units[(size_t)u * 64 + lane] = t;
        const int32_t m = wave_min_i32(t);
        if (lane == 0) unit_min[u] = m;
    }
}

// ---- what a table says about candidates (once per table)
//
// For BAND_THRESHOLDS values of t_max, from the largest latency down: a candidate takes what is known of the next
// threshold that is not below it, whose filter leaves every term of its own.
//   * Windows.  A plan has a stage of the layers k .. on d devices behind it only if the layers from k on need no
//     more than d under the filter and those in front of k leave as many.  With t_max at the low end, where most
//     layers are run, few device counts are left: 1 to 16 a block of eight layers where the smallest
//     t_max with a plan takes all of 64 devices.
//   * Front costs.  P(k, d): the least sum of stages that cover the k layers in front on d devices, with the least
//     t_intra over the number of stages behind them.  F(s, k, d) + P(k, D - d) bounds every plan that goes on from
//     there, so a candidate is finished once no cell of layer s gets below what it has (64 layers on 8 x 8 of
//     dense layers, t_max at the 5 % quantile: after 4 layers, 9 with the least F of more stages and no filter).
// And without a filter: the least largest stage (no plan below that t_max), and the lowest threshold whose least plan
// is that without a filter (from there on F hardly changes).  least[k][i][q]: q padded (SP).
// Windows of one threshold.  `need`: fewest devices of each stage; then wave 0 goes through the layers from the front
// and wave 1 from the back.  NX: layers / 64, at least.
template <int NX>
__device__ __forceinline__ void band_find_windows(const int32_t *__restrict__ least, const int32_t *__restrict__ sizes,
                                                  int K, int D, int S, int SP, int32_t c, uint16_t *need, int32_t *windows)
{
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = K | 1;                          // (odd: a column is read as fast as a row)
    for (int x = tid; x < K * K; x += blockDim.x) {
        const int4 *row = (const int4 *)(least + (size_t)x * SP);
        int m = 1 << 14;
        for (int q = 0; q < S; q += 4) {
            const int4 t = row[q >> 2];
            if (t.x <= c) m = min(m, sizes[q]);
            if (t.y <= c) m = min(m, sizes[min(q + 1, S - 1)]);
            if (t.z <= c) m = min(m, sizes[min(q + 2, S - 1)]);
            if (t.w <= c) m = min(m, sizes[min(q + 3, S - 1)]);
        }
        need[(x / K) * KS + x % K] = (uint16_t)m;  // (the stage of layers x / K .. x % K)
    }
    __syncthreads();
    if (wid >= 2) return;
    const bool front = wid == 0;
    int v[NX];                                     // front: fewest devices of layers 0 .. k - 1, k = 64 x + lane; back: of k .. K - 1
#pragma unroll
    for (int x = 0; x < NX; ++x) v[x] = front && x == 0 && lane == 0 ? 0 : 1 << 20;
    int far = 0;
    constexpr int Y = 8;                           // rows read ahead
    for (int y0 = 0; y0 < K; y0 += Y) {
        int m[Y][NX];
#pragma unroll
        for (int y = 0; y < Y; ++y) {
            const int i = front ? min(y0 + y, K - 1) : max(K - 1 - y0 - y, 0);     // stages that begin (end) with layer i
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const int k = WAVE * x + lane - (front ? 1 : 0), at = max(0, min(k, K - 1));
                const int n = need[front ? i * KS + at : at * KS + i];
                m[y][x] = k < 0 ? 1 << 20 : n;
            }
        }
#pragma unroll
        for (int y = 0; y < Y; ++y) {
            if (y0 + y >= K) break;
            const int i = front ? y0 + y : K - 1 - y0 - y;
            if (front) {
#pragma unroll
                for (int x = 0; x < NX; ++x)
                    if (x == 0 || i >= WAVE * x) far = __builtin_amdgcn_readlane(v[x], i & 63);
            }
#pragma unroll
            for (int x = 0; x < NX; ++x) v[x] = min(v[x], far + m[y][x]);
            if (!front) {
#pragma unroll
                for (int x = 0; x < NX; ++x)
                    if (x == 0 || i >= WAVE * x) far = __builtin_amdgcn_readlane(v[x], i & 63);
            }
        }
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        int m = WAVE * x + lane < K ? v[x] : 1 << 20;      // the least of the block's eight
        m = min(m, dpp_mov<0xB1>(m));
        m = min(m, dpp_mov<0x4E>(m));
        m = min(m, dpp_mov<0x141>(m));
        const int b = 8 * x + (lane >> 3);
        if ((lane & 7) == 0 && b < 32) windows[(front ? 32 : 0) + b] = front ? max(0, D - m) : min(m, D + 1);
    }
    for (int b = 8 * NX + lane; b < 32; b += WAVE) windows[(front ? 32 : 0) + b] = front ? 0 : D + 1;
}

// Blocks [0, BAND_THRESHOLDS): P, then as many for Q, then the least largest stage, then windows.
// fronts[j][k][RS]: P(k, D - d) at d - 1 (+infinity where no layer or no device is in front); backs[j][k][RS]: Q(k, d) at d - 1;
// totals[j]: P(K, D), and the least largest stage behind the last.
// A plan of one stage (latency as it is) bounds every sum, so no longer stage is looked at, whatever the filter.
// Bound by the sums of the highest thresholds, whose filter leaves every stage: 64 layers on 8 x 8 92 us, 128 layers 300, 48 on 32 x 8
// 360 (P alone, a chain of rows that all waves wait for: 105, 320 and 420).  The windows beside them cost nothing: done twice, the same.
template <int W, int NH>
__global__ __launch_bounds__(WAVE * FRONT_WAVES) void band_thresholds_kernel(FrontTable ft, FrontTable ft_back, const int32_t *__restrict__ table,
                                                                              BandShapes bs, int K, int D, int32_t max_finite,
                                                                              int32_t *__restrict__ fronts, int32_t *__restrict__ backs,
                                                                              int32_t *__restrict__ totals, int32_t *__restrict__ plans,
                                                                              int32_t *__restrict__ windows, int32_t *graph_used,
                                                                              const int32_t *__restrict__ there)
{
    if (there && *there) return;
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];
    constexpr int RS = WAVE * W;
    const int S = bs.S, R = D + 2, what = blockIdx.x / BAND_THRESHOLDS, j = blockIdx.x - what * BAND_THRESHOLDS;
    const FrontLds l = front_lds(lds, K, D, ft.NG, W);
    if (what < 2) {
        const int32_t c = min(band_threshold(max_finite, j), front_single(table, bs, K, D));
        front_costs<W, FRONT_WAVES, NH, false>(what ? ft_back : ft, K, D, S, c, l);
        int32_t *const out = (what ? backs : fronts) + (size_t)j * K * RS;
        for (int x = threadIdx.x; x < K * RS; x += blockDim.x) {
            const int k = x / RS, d = x - k * RS + 1;
            out[x] = what ? (d <= D ? l.P[(K - k) * R + 1 + d] : DEV_INF) : k >= 1 && d < D ? l.P[k * R + 1 + D - d] : DEV_INF;
        }
        if (what) return;
        if (threadIdx.x == 0) totals[j] = l.P[K * R + 1 + D];
        front_plan(ft, table, bs, K, D, c, l.P, plans + 2 * j);
        return;
    }
    if (blockIdx.x == 2 * BAND_THRESHOLDS) {
        front_costs<W, FRONT_WAVES, NH, true>(ft, K, D, S, DEV_INF - 1, l);
        if (threadIdx.x == 0) {
            totals[BAND_THRESHOLDS] = l.P[K * R + 1 + D];
            plans[2 * BAND_THRESHOLDS] = 0;        // (band_bounds counts there)
            if (graph_used) *graph_used = 0;       // (sparse_graph_kernel counts there)
        }
        return;
    }
    const int w = blockIdx.x - 2 * BAND_THRESHOLDS - 1, SP = front_padded(S);
    const int32_t c = band_threshold(max_finite, w);
    if (K <= 64) band_find_windows<1>(ft.least, bs.sizes, K, D, S, SP, c, (uint16_t *)lds, windows + 64 * w);
    else if (K <= 128) band_find_windows<2>(ft.least, bs.sizes, K, D, S, SP, c, (uint16_t *)lds, windows + 64 * w);
    else band_find_windows<4>(ft.least, bs.sizes, K, D, S, SP, c, (uint16_t *)lds, windows + 64 * w);
}

size_t front_lds_bytes(int K, int D, int S)
{
    return (size_t)front_lds(nullptr, K, D, front_groups(S), D <= 64 ? 1 : D <= 128 ? 2 : 4).ints * 4;
}

// What front costs are found from, laid out when the table is (a recorded solve launches only what depends on the bounds not being
// there).  work: front_least_ints; front: front_table_ints
hipError_t launch_front_table(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t *work, int32_t *front)
{
    const int K = p.K, SP = front_padded(b.S);
    const FrontTable ft = front_table(work, front, K, b.S, b.sizes, false);
    hipLaunchKernelGGL(front_least_kernel, dim3(std::min((K * K * SP + 255) / 256, 16384)), dim3(256), 0, st, table, K, p.Smax, b, SP,
                       work, (uint8_t *)ft.run);
    hipLaunchKernelGGL(front_units_kernel, dim3(std::min((front_units(K, b.S) + 3) / 4, 8192), 2), dim3(256), 0, st, work, K, b.S, SP,
                       (int32_t *)ft.units);
    return hipGetLastError();
}

// behind launch_front_table of the same table
hipError_t launch_front_thresholds(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                                   const int32_t *work, const int32_t *front, int32_t *fronts, int32_t *backs, int32_t *totals,
                                   int32_t *plans, int32_t *windows, int32_t *graph_used, const int32_t *asked)
{
    const int K = p.K, D = p.D;
    const FrontTable ft = front_table(work, front, K, b.S, b.sizes, false), ft_back = front_table(work, front, K, b.S, b.sizes, true);
    const size_t lds = std::max(front_lds_bytes(K, D, b.S), (size_t)2 * K * (K | 1));
    const auto kernel = D > 128 ? band_thresholds_kernel<4, 0> : D > 64 ? band_thresholds_kernel<2, 0> : b.S > 16 ? band_thresholds_kernel<1, 0> :
                        b.S > 12 ? band_thresholds_kernel<1, 4> : b.S > 8 ? band_thresholds_kernel<1, 3> : band_thresholds_kernel<1, 2>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(3 * BAND_THRESHOLDS + 1), dim3(WAVE * FRONT_WAVES), lds, st, ft, ft_back, table, b, K, D,
                       max_finite, fronts, backs, totals, plans, windows, graph_used, asked);
    return hipGetLastError();
}

}  // namespace alpa
