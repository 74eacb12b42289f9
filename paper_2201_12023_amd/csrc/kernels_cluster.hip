// Operator clustering on the device (Sec. 5.2, performance optimisation #2, Eq. 6):
//   G(n, r) = min over 1 <= i <= n with FLOP(o_i..o_n) <= cap of max{G(i-1, r-1), C(i, n)},
// C(i, n) = bytes that o_i..o_n receive from o_1..o_{i-1}; ties go to the smaller sum of squared
// per-layer FLOP (carried as V(n, r)), then to the smaller i.
//
// FLOP figures are non-negative, so the feasible i of an n are the last win(n) ones, found by bisection on
// the FLOP prefix sums, and only a band of C is ever read.  It is kept by distance, band[j][n] = C(n - j, n),
// j < max win: with w(u, v) the bytes of the edges u -> v,
//   in(j, v) = bytes into v from before v - j = in(v) - sum over d <= j of w(v - d, v)   (a prefix along j),
//   C(i, n)  = sum over v = i..n of in(v - i, v)                                 (a running sum along a diagonal),
// both with neighbouring operators in neighbouring lanes.  (The full matrix took six passes over 8 K^2
// bytes: 240 of 790 us at 3002 operators; the band takes 20.)
//
// The recurrence over r is one launch for up to ROWS_PER_LAUNCH values of r (cluster_rows_kernel): a workgroup
// owns a tile of consecutive n, with 16 lanes per n that share its candidates, whose C values stay in registers; row
// r - 1 of its own tile is in LDS, and the rows of the tiles in front come through memory.
#include "internal.hpp"

namespace alpa {

constexpr int CL_THREADS = 1024;
constexpr int CL_LANES = 16;           // lanes per prefix length n
constexpr int CL_TILE = CL_THREADS / CL_LANES;     // prefix lengths per workgroup
constexpr int CL_KEEP = 8;             // candidates per lane whose C and squared FLOP are kept in registers
constexpr int ROWS_PER_LAUNCH = 128;
constexpr int64_t NOT_YET = -1;        // no value of a row is negative

// pf[x] = FLOP of operators 0..x-1 (int64); win[n] = number of feasible first operators of a layer that ends
// with the n-th (1-based); meta[0] = the largest of them (at least 1), meta[1] = work counter, meta[2] = a wait
// has run out.  One block.
__global__ __launch_bounds__(CL_THREADS) void cluster_prefix_kernel(
    const int32_t *__restrict__ flop, int K, int64_t cap, const int64_t *__restrict__ ctl,
    int64_t *__restrict__ pf, int32_t *__restrict__ win, int64_t *__restrict__ tot, int32_t *__restrict__ meta)
{
    extern __shared__ int64_t sh[];                  // [K + 1] prefix sums
    __shared__ int64_t part[CL_THREADS];
    __shared__ int sh_max;
    // Bound computed on the device (cluster_check_kernel).  Inputs that it has refused have no feasible first
    // operator anywhere: with a negative figure a row value could be any number, NOT_YET among them.
    const bool refused = ctl && ctl[0] != 0;
    if (ctl) cap = ctl[1];
    const int t = threadIdx.x;
    const int per = (K + CL_THREADS - 1) / CL_THREADS;
    const int lo = min(K, t * per), hi = min(K, lo + per);
    int64_t s = 0;
    for (int x = lo; x < hi; ++x) s += flop[x];
    part[t] = s;
    if (t == 0) { sh_max = 1; sh[0] = 0; }
    __syncthreads();
    for (int off = 1; off < CL_THREADS; off <<= 1) {
        const int64_t o = (t >= off) ? part[t - off] : 0;
        __syncthreads();
        part[t] += o;
        __syncthreads();
    }
    int64_t run = part[t] - s;
    for (int x = lo; x < hi; ++x) {
        run += flop[x];
        sh[x + 1] = run;
    }
    __syncthreads();
    int widest = 1;
    for (int n = t; n <= K; n += CL_THREADS) {
        pf[n] = sh[n];
        if (n < K) tot[n] = 0;
        // smallest x = i - 1 in [0, n] with pf[n] - pf[x] <= cap (n itself: nothing fits)
        const int64_t need = sh[n] - cap;
        int a = 0, b = n;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (sh[mid] >= need) b = mid; else a = mid + 1;
        }
        const int feasible = refused ? 0 : n - a;
        win[n] = feasible;
        widest = max(widest, feasible);
    }
    atomicMax(&sh_max, widest);
    __syncthreads();
    if (t == 0) { meta[0] = sh_max; meta[1] = 0; meta[2] = 0; }
}

__global__ void cluster_zero_band_kernel(int64_t *__restrict__ band, int K, const int32_t *__restrict__ meta)
{
    const long long n = (long long)meta[0] * K;
    for (long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x; x < n;
         x += (long long)gridDim.x * blockDim.x)
        band[x] = 0;
}

// band[v - u][v] += bytes(u -> v) inside the band; tot[v] += bytes of every edge into v
__global__ void cluster_edges_kernel(const int32_t *__restrict__ src, const int32_t *__restrict__ dst,
                                     const int64_t *__restrict__ nbytes, int E, int K,
                                     int64_t *__restrict__ band, int64_t *__restrict__ tot,
                                     const int32_t *__restrict__ meta)
{
    const int width = meta[0];
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < E; e += gridDim.x * blockDim.x) {
        const int u = src[e], v = dst[e];
        // callers with host arrays have checked this already; with device arrays the check
        // kernel reports such an edge, and here it must not be written
        if (u < 0 || v >= K || u >= v) continue;
        atomicAdd((unsigned long long *)&tot[v], (unsigned long long)nbytes[e]);
        if (v - u < width)
            atomicAdd((unsigned long long *)&band[(size_t)(v - u) * K + v], (unsigned long long)nbytes[e]);
    }
}

// band[j][v] = bytes into v from operators before v - j, in place: a thread per v
__global__ __launch_bounds__(64) void cluster_band_in_kernel(int64_t *__restrict__ band,
                                                             const int64_t *__restrict__ tot, int K,
                                                             const int32_t *__restrict__ meta)
{
    const int v = blockIdx.x * 64 + threadIdx.x;
    if (v >= K) return;
    const int width = min(meta[0], v + 1);
    int64_t run = tot[v];
    int64_t *p = band + v;
    int j = 0;
    for (; j + 8 <= width; j += 8) {                 // loads ahead of the chain of sums
        int64_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(size_t)(j + u) * K];
#pragma unroll
        for (int u = 0; u < 8; ++u) { run -= x[u]; p[(size_t)(j + u) * K] = run; }
    }
    for (; j < width; ++j) { run -= p[(size_t)j * K]; p[(size_t)j * K] = run; }
}

// band[j][i + j] = C(i, i + j), in place: a thread per first operator i
__global__ __launch_bounds__(64) void cluster_band_sum_kernel(int64_t *__restrict__ band, int K,
                                                              const int32_t *__restrict__ meta)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= K) return;
    const int width = min(meta[0], K - i);
    int64_t run = 0;
    int64_t *p = band + i;
    const size_t step = (size_t)K + 1;
    int j = 0;
    for (; j + 8 <= width; j += 8) {
        int64_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(j + u) * step];
#pragma unroll
        for (int u = 0; u < 8; ++u) { run += x[u]; p[(j + u) * step] = run; }
    }
    for (; j < width; ++j) { run += p[j * step]; p[j * step] = run; }
}

// Rows of one launch: row 0 is the row in front (the empty prefix alone for the first launch, else the
// last row of the launch before), the others are not there yet.  EXACT rows hold W in V.
__global__ void cluster_begin_rows_kernel(int64_t *__restrict__ G, int64_t *__restrict__ V, int K, int rows,
                                          int first, int exact, int last_row, int32_t *__restrict__ meta)
{
    const size_t ld = (size_t)K + 1;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x <= K; x += gridDim.x * blockDim.x) {
        if (first) {
            if (!exact) G[x] = x == 0 ? 0 : INF_I64;
            V[x] = (exact && x != 0) ? INF_I64 : 0;
        } else {
            if (!exact) G[x] = G[last_row * ld + x];
            V[x] = V[last_row * ld + x];
        }
        // (row 0 is written by the same thread, from a row that only this thread touches)
        for (int r = 1; r <= rows; ++r) {
            if (!exact) G[r * ld + x] = NOT_YET;
            V[r * ld + x] = NOT_YET;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) meta[1] = 0;
}

struct Lex {                    // (G, V, i): smaller is better, component by component
    int64_t g, v;
    int i;
};
__device__ __forceinline__ bool lex_less(const Lex &a, const Lex &b)
{
    return a.g < b.g || (a.g == b.g && (a.v < b.v || (a.v == b.v && a.i < b.i)));
}
template <int CTRL>
__device__ __forceinline__ void lex_step(Lex &a)
{
    const Lex o{dpp_mov64<CTRL>(a.g), dpp_mov64<CTRL>(a.v), dpp_mov<CTRL>(a.i)};
    if (lex_less(o, a)) a = o;
}

// The value at p once it is there.  Every wait of a call that has the work memory to itself ends by itself (see
// cluster_rows_kernel); what another call overwrites may never come, so after max_spins looks, or once some
// wait has run out (*lost), the caller goes on without it and the call reports it.  (A clock in the place of
// the count is 2 % of the whole call.)
__device__ __forceinline__ int64_t await(const int64_t *p, int32_t *lost, unsigned max_spins)
{
    int64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (unsigned spin = 0; v == NOT_YET; ++spin) {
        if (spin >= max_spins ||
            (spin % 64 == 63 && __hip_atomic_load(lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            __hip_atomic_store(lost, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return INF_I64;
        }
        __builtin_amdgcn_s_sleep(1);
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return v;
}

// Rows 1..rows of this launch, 64 prefix lengths to a workgroup.  Bound by the way of a value from one
// workgroup to the next (2.5 us a row at 3002 operators; a launch per row took 5.8).  512 prefix lengths to
// a workgroup, two lanes each, need no such way up to 512 operators, but take 3 us a row to compute.
// A tile reads rows of tiles in front of it only, and tiles are handed out in order, so the workgroup
// that a wait is for has always started and waits itself only for tiles further in front: every
// wait ends.  A value is its own signal (NOT_YET until it is there), so no fence is needed.
// EXACT (the variance tie-break over whole clusterings): with G* = G(K, L) in *gstar_p,
//   W(n, r) = min over the feasible i with C(i, n) <= G* of W(i-1, r-1) + FLOP(o_i..o_n)^2, lowest i on ties.
template <bool EXACT>
__global__ __launch_bounds__(CL_THREADS) void cluster_rows_kernel(
    const int64_t *__restrict__ band, const int64_t *__restrict__ pf, const int32_t *__restrict__ win, int K,
    int rows, int64_t *G, int64_t *V, int32_t *__restrict__ arg, int32_t *meta,
    const int64_t *__restrict__ gstar_p, unsigned max_spins)
{
    constexpr int T = CL_TILE, GL = CL_LANES, KEEP = CL_KEEP;
    extern __shared__ int64_t sh[];
    __shared__ int sh_tile;
    if (threadIdx.x == 0) sh_tile = atomicAdd(&meta[1], 1);
    __syncthreads();
    const int n0 = sh_tile * T;                      // the tile: prefix lengths n0 + 1 .. n0 + T
    if (n0 >= K) return;
    const int g = threadIdx.x % GL, nl = threadIdx.x / GL;
    const int n = n0 + 1 + nl;
    const int base = max(0, n0 - meta[0] + 1);       // first prefix length that the tile reads
    const int halo = n0 + 1 - base;                  // base .. n0 come from tiles in front
    const int size = halo + T;
    int64_t *sG = sh, *sV = sh + size, *sP = sh + 2 * size;
    const size_t ld = (size_t)K + 1;
    for (int x = threadIdx.x; x < size; x += CL_THREADS) {
        const int m = min(base + x, K);
        sP[x] = pf[m];
        if (!EXACT) sG[x] = G[m];
        sV[x] = V[m];
    }
    // (no further back than the tile reads, whatever another call may have left in `win`)
    const int width = n <= K ? min(win[n], n - base) : 0;
    const int64_t pn = pf[min(n, K)];
    const int64_t gstar = EXACT ? *gstar_p : 0;
    __syncthreads();
    // FLOP(o_i..o_n)^2, i = n - j (a layer's FLOP fits 31 bits)
    auto squared = [&](int j) {
        const uint32_t f = (uint32_t)(pn - sP[n - 1 - j - base]);
        return (int64_t)((uint64_t)f * f);
    };
    int64_t keep_c[KEEP], keep_f[KEEP];
#pragma unroll
    for (int u = 0; u < KEEP; ++u) {
        const int j = g + u * GL;
        keep_c[u] = j < width ? band[(size_t)j * K + n - 1] : 0;
        keep_f[u] = j < width ? squared(j) : 0;
    }
    for (int r = 1; r <= rows; ++r) {
        if (r > 1)
            for (int x = threadIdx.x; x < halo; x += CL_THREADS) {
                const int m = base + x;
                // G(0, r) of a positive number of layers is infinite; nobody owns it
                if (!EXACT) sG[x] = m == 0 ? INF_I64 : await(&G[(r - 1) * ld + m], &meta[2], max_spins);
                sV[x] = m == 0 ? (EXACT ? INF_I64 : 0) : await(&V[(r - 1) * ld + m], &meta[2], max_spins);
            }
        __syncthreads();
        Lex best{INF_I64, 0, 0};
        auto term = [&](int j, int64_t c, int64_t ff) {
            const int x = n - 1 - j - base;          // prefix length i - 1, i = n - j
            Lex cur;
            if (EXACT) {
                const int64_t wp = sV[x];
                if (gstar == INF_I64 || wp == INF_I64 || c > gstar) return;
                cur = Lex{wp + ff, 0, n - j};
            } else {
                const int64_t gp = sG[x];
                if (gp == INF_I64) return;
                cur = Lex{gp > c ? gp : c, sV[x] + ff, n - j};
            }
            if (lex_less(cur, best)) best = cur;
        };
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            const int j = g + u * GL;
            if (j < width) term(j, keep_c[u], keep_f[u]);
        }
        for (int j = g + KEEP * GL; j < width; j += GL)
            term(j, band[(size_t)j * K + n - 1], squared(j));
        lex_step<0xB1>(best);                        // the n's 16 lanes: neighbours, pairs, quads, halves of a row
        lex_step<0x4E>(best);
        lex_step<0x141>(best);
        lex_step<0x140>(best);
        if (best.g == INF_I64) { best.v = 0; best.i = 0; }
        __syncthreads();                             // the row in front has been read
        if (g == 0 && n <= K) {
            const int64_t v = EXACT ? best.g : best.v;
            if (!EXACT) sG[halo + nl] = best.g;
            sV[halo + nl] = v;
            if (!EXACT) __hip_atomic_store(&G[r * ld + n], best.g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&V[r * ld + n], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            arg[(r - 1) * ld + n] = best.i;
        }
        if (r > 0 && threadIdx.x == 0 && n0 == 0) {  // G(0, r), for the row that the next launch starts from
            if (!EXACT) G[r * ld] = INF_I64;
            V[r * ld] = EXACT ? INF_I64 : 0;
            arg[(r - 1) * ld] = 0;
        }
    }
}

// *keep = G(K, L) of the first run (the second one does not write the G rows)
__global__ void cluster_keep_kernel(const int64_t *__restrict__ G, int64_t *__restrict__ keep) { *keep = *G; }

// Argument checks for device-resident inputs (what alpa_cluster_layers does on the host):
// ctl[0] = 0, ALPA_DP_EINVAL (-1: negative figure, bad edge) or ALPA_DP_EOVERFLOW (-2: total FLOP
// >= 2^31, total * L >= 2^42, edge sizes adding up to >= 2^62); ctl[1] = the FLOP bound per
// layer, floor((10^6 + delta_ppm) * total / (L * 10^6)).  One block.
__global__ __launch_bounds__(1024) void cluster_check_kernel(
    const int32_t *__restrict__ flop, int K, const int32_t *__restrict__ src,
    const int32_t *__restrict__ dst, const int64_t *__restrict__ nbytes, int E, int L,
    int delta_ppm, int64_t *__restrict__ ctl)
{
    __shared__ unsigned long long sh_flop, sh_bytes;
    __shared__ int sh_bad, sh_over;
    const int t = threadIdx.x;
    if (t == 0) { sh_flop = 0; sh_bytes = 0; sh_bad = 0; sh_over = 0; }
    __syncthreads();
    constexpr unsigned long long LIM = 1ull << 62;
    unsigned long long f = 0, b = 0;
    int bad = 0, over = 0;
    for (int k = t; k < K; k += 1024) {
        const int32_t v = flop[k];
        if (v < 0) bad = 1; else f += (unsigned long long)v;        // < 2^31 * 4 per thread
    }
    for (int e = t; e < E; e += 1024) {
        const int u = src[e], v = dst[e];
        const int64_t n = nbytes[e];
        if (u < 0 || v >= K || u >= v || n < 0) { bad = 1; continue; }
        if ((unsigned long long)n >= LIM) over = 1;
        b = min(LIM, b + min(LIM, (unsigned long long)n));         // saturating: stays <= 2^62
    }
    atomicAdd(&sh_flop, f);
    if (bad) atomicOr(&sh_bad, 1);
    if (over) atomicOr(&sh_over, 1);
    __syncthreads();
    // the byte total, saturating, one thread after the other (1024 partial sums <= 2^62 each
    // would wrap an unsigned 64-bit add)
    for (int turn = 0; turn < 1024; turn += WAVE) {
        if (t >= turn && t < turn + WAVE) {
            unsigned long long x = b;
            for (int off = 32; off >= 1; off >>= 1) {
                const unsigned long long o =
                    (unsigned long long)i64_from(__shfl_xor(lo32((int64_t)x), off, 64),
                                                 __shfl_xor(hi32((int64_t)x), off, 64));
                x = min(LIM, x + o);
            }
            if ((t & (WAVE - 1)) == 0) sh_bytes = min(LIM, sh_bytes + x);
        }
        __syncthreads();
    }
    if (t == 0) {
        const unsigned long long total = sh_flop;
        int64_t status = 0;
        if (sh_bad) status = -1;
        else if (total >= (1ull << 31) || total * (unsigned long long)L >= (1ull << 42) ||
                 sh_over || sh_bytes >= LIM) status = -2;
        ctl[0] = status;
        ctl[1] = status ? 0
                        : (int64_t)(((1000000ull + (unsigned long long)delta_ppm) * total) /
                                    ((unsigned long long)L * 1000000ull));
    }
}

// out[0] = G(K, L), out[1] = V(K, L); first_op[0..L] by walking arg back (one thread).  out[2] = 0, or ctl[0], the
// status of the argument checks (device-resident inputs), or -4 (ALPA_DP_EHIP) if a wait has run out; "no
// clustering" is reported if that is not 0.
__global__ void cluster_walk_kernel(const int64_t *__restrict__ G, const int64_t *__restrict__ V,
                                    const int32_t *__restrict__ arg, int K, int L,
                                    const int64_t *__restrict__ ctl, const int32_t *__restrict__ meta,
                                    int64_t *__restrict__ out, int32_t *__restrict__ first_op)
{
    // G: G(K, L); V: the sum of squares that goes with it (exact mode: W(K, L))
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const int64_t status = ctl && ctl[0] != 0 ? ctl[0] : meta[2] != 0 ? -4 : 0;
    out[2] = status;
    const int64_t g = status != 0 ? INF_I64 : *G;
    out[0] = g;
    out[1] = g == INF_I64 ? 0 : *V;
    if (g == INF_I64) {
        for (int r = 0; r <= L; ++r) first_op[r] = -1;
        return;
    }
    int n = K;
    first_op[L] = K;
    for (int r = L; r >= 1; --r) {
        const int i = arg[(size_t)(r - 1) * (K + 1) + n];
        n = min(max(i - 1, 0), K);                   // (i is in 1..n unless another call wrote here)
        first_op[r - 1] = n;
    }
}

template <bool EXACT>
static hipError_t launch_rows(hipStream_t st, const ClusterWork &w, int K, int rows, int width, int32_t *arg,
                              unsigned max_spins)
{
    constexpr int T = CL_TILE;
    const size_t lds = (size_t)3 * (std::min(width, K) + T + 1) * sizeof(int64_t);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)cluster_rows_kernel<EXACT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((cluster_rows_kernel<EXACT>), dim3((K + T - 1) / T), dim3(CL_THREADS), lds, st, w.band,
                       w.pf, w.win, K, rows, w.G, w.V, arg, w.meta, w.keep, max_spins);
    return hipGetLastError();
}

template <bool EXACT>
static hipError_t launch_run(hipStream_t st, const ClusterWork &w, int K, int L, int width, int32_t *arg,
                             unsigned max_spins)
{
    const size_t ld = (size_t)K + 1;
    int done = 0, last = 0;
    while (done < L) {
        const int rows = std::min(ROWS_PER_LAUNCH, L - done);
        hipLaunchKernelGGL(cluster_begin_rows_kernel, dim3((K + 64) / 64), dim3(64), 0, st, w.G, w.V, K, rows,
                           done == 0 ? 1 : 0, EXACT ? 1 : 0, last, w.meta);
        const hipError_t e = launch_rows<EXACT>(st, w, K, rows, width, arg + done * ld, max_spins);
        if (e != hipSuccess) return e;
        done += rows;
        last = rows;
    }
    return hipSuccess;
}

hipError_t launch_cluster(hipStream_t st, const int32_t *flop, const int32_t *src,
                          const int32_t *dst, const int64_t *nbytes, int E, int K, int L,
                          int64_t cap, int width, const ClusterWork &w, int64_t *out,
                          int32_t *first_op, int64_t *ctl, int delta_ppm, int exact,
                          unsigned max_spins)
{
    if (ctl)
        hipLaunchKernelGGL(cluster_check_kernel, dim3(1), dim3(1024), 0, st, flop, K, src, dst,
                           nbytes, E, L, delta_ppm, ctl);
    hipLaunchKernelGGL(cluster_prefix_kernel, dim3(1), dim3(CL_THREADS), ((size_t)K + 1) * 8, st, flop, K, cap,
                       (const int64_t *)ctl, w.pf, w.win, w.tot, w.meta);
    const long long cells = (long long)width * K;
    hipLaunchKernelGGL(cluster_zero_band_kernel, dim3((unsigned)std::min<long long>((cells + 1023) / 1024, 1024)),
                       dim3(256), 0, st, w.band, K, w.meta);
    if (E > 0)
        hipLaunchKernelGGL(cluster_edges_kernel, dim3((E + 255) / 256), dim3(256), 0, st, src, dst,
                           nbytes, E, K, w.band, w.tot, w.meta);
    hipLaunchKernelGGL(cluster_band_in_kernel, dim3((K + 63) / 64), dim3(64), 0, st, w.band, w.tot, K, w.meta);
    hipLaunchKernelGGL(cluster_band_sum_kernel, dim3((K + 63) / 64), dim3(64), 0, st, w.band, K, w.meta);
    hipError_t e = launch_run<false>(st, w, K, L, width, w.arg, max_spins);
    if (e != hipSuccess) return e;
    const size_t ld = (size_t)K + 1;
    const size_t end = (size_t)((L - 1) % ROWS_PER_LAUNCH + 1) * ld + K;   // (K, L) in the last launch's rows
    if (exact) {
        hipLaunchKernelGGL(cluster_keep_kernel, dim3(1), dim3(1), 0, st, w.G + end, w.keep);
        e = launch_run<true>(st, w, K, L, width, w.arg, max_spins);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(cluster_walk_kernel, dim3(1), dim3(WAVE), 0, st, exact ? w.keep : w.G + end, w.V + end,
                       w.arg, K, L, (const int64_t *)ctl, w.meta, out, first_op);
    return hipGetLastError();
}

// int64 units of the work memory, and its parts
size_t cluster_work_i64(int K, int L, int width)
{
    const size_t ld = (size_t)K + 1, rows = (size_t)std::min(L, ROWS_PER_LAUNCH) + 1;
    return (size_t)width * K + 2 * rows * ld + ld + K + 8 + (ld + (size_t)L * ld + 3) / 2;
}

ClusterWork cluster_work(int64_t *base, int K, int L, int width)
{
    const size_t ld = (size_t)K + 1, rows = (size_t)std::min(L, ROWS_PER_LAUNCH) + 1;
    ClusterWork w{};
    w.keep = base;
    w.meta = (int32_t *)(base + 1);
    w.pf = base + 8;
    w.tot = w.pf + ld;
    w.G = w.tot + K;
    w.V = w.G + rows * ld;
    w.band = w.V + rows * ld;
    w.win = (int32_t *)(w.band + (size_t)width * K);
    w.arg = w.win + ld;
    return w;
}

// Largest number of feasible first operators over the operators, as cluster_prefix_kernel finds it (host
// arrays; the FLOP figures are non-negative, so both ends of the window only move forward)
int cluster_band_width(const int32_t *flop, int K, int64_t cap)
{
    int64_t sum = 0;
    int first = 0, widest = 1;
    for (int n = 0; n < K; ++n) {
        sum += flop[n];
        while (sum > cap) sum -= flop[first++];
        widest = std::max(widest, n + 1 - first);
    }
    return widest;
}

}  // namespace alpa
