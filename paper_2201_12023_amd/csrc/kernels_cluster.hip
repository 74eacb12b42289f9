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
// owns a tile of consecutive n, with 8 or 16 lanes per n that share its candidates, whose C values stay in registers; row
// r - 1 of its own tile is in LDS, and the rows of the tiles in front come through memory.
#include "internal.hpp"

#include <type_traits>

namespace alpa {

constexpr int CL_THREADS = 1024;
// A workgroup that computes rows: LANES to a prefix length n, FETCH waves that fetch what is in front, TILE prefix lengths, and KEEP
// candidates per lane whose C and squared FLOP are kept in registers.
template <int L, int N_THREADS, int F>
struct RowForm {
    static constexpr int LANES = L, THREADS = N_THREADS, FETCH = F, TILE = (N_THREADS - F * WAVE) / L, KEEP = 16;
};
constexpr int ROWS_PER_LAUNCH = 128;
constexpr int64_t NOT_YET = -1;        // no value of a row is negative

// Argument checks for device-resident inputs (what alpa_cluster_layers does on the host):
// ctl[0] = 0, ALPA_DP_EINVAL (-1: negative figure, bad edge) or ALPA_DP_EOVERFLOW (-2: total FLOP
// >= 2^31, total * L >= 2^42, edge sizes adding up to >= 2^62); ctl[1] = the FLOP bound per
// layer, floor((10^6 + delta_ppm) * total / (L * 10^6)).  One block.
// (ends with a barrier; whether they are refused, and the bound)
struct ClusterInputs {
    const int32_t *src, *dst;
    const int64_t *nbytes;
    int E, L, delta_ppm;
};
__device__ __forceinline__ bool cluster_check(const int32_t *__restrict__ flop, int K, const ClusterInputs &in, int64_t *__restrict__ ctl,
                                              int64_t &cap)
{
    const int32_t *__restrict__ const src = in.src, *__restrict__ const dst = in.dst;
    const int64_t *__restrict__ const nbytes = in.nbytes;
    const int E = in.E, L = in.L;
    __shared__ int64_t sh_ctl[2];
    __shared__ unsigned long long sh_flop[CL_THREADS / WAVE], sh_bytes[CL_THREADS / WAVE];
    __shared__ int sh_bad, sh_over;
    const int t = threadIdx.x;
    if (t == 0) { sh_bad = 0; sh_over = 0; }
    __syncthreads();
    constexpr unsigned long long LIM = 1ull << 62;
    unsigned long long f = 0, b = 0;
    int bad = 0, over = 0;
    for (int k = t; k < K; k += CL_THREADS) {
        const int32_t v = flop[k];
        if (v < 0) bad = 1; else f += (unsigned long long)v;        // < 2^31 * 4 per thread
    }
    for (int e = t; e < E; e += CL_THREADS) {
        const int u = src[e], v = dst[e];
        const int64_t n = nbytes[e];
        if (u < 0 || v >= K || u >= v || n < 0) { bad = 1; continue; }
        if ((unsigned long long)n >= LIM) over = 1;
        b = min(LIM, b + min(LIM, (unsigned long long)n));         // saturating: stays <= 2^62
    }
    if (bad) atomicOr(&sh_bad, 1);
    if (over) atomicOr(&sh_over, 1);
    // the byte total saturates at every sum (1024 partial ones of up to 2^62 would wrap an unsigned 64-bit add)
    for (int off = 32; off >= 1; off >>= 1) {
        f += __shfl_xor(f, off, WAVE);
        b = min(LIM, b + __shfl_xor(b, off, WAVE));
    }
    if ((t & (WAVE - 1)) == 0) { sh_flop[t / WAVE] = f; sh_bytes[t / WAVE] = b; }
    __syncthreads();
    if (t == 0) {
        unsigned long long total = 0, bytes = 0;
        for (int w = 0; w < CL_THREADS / WAVE; ++w) {
            total += sh_flop[w];
            bytes = min(LIM, bytes + sh_bytes[w]);
        }
        int64_t status = 0;
        if (sh_bad) status = -1;
        else if (total >= (1ull << 31) || total * (unsigned long long)L >= (1ull << 42) ||
                 sh_over || bytes >= LIM) status = -2;
        ctl[0] = sh_ctl[0] = status;
        ctl[1] = sh_ctl[1] = status ? 0
                        : (int64_t)(((1000000ull + (unsigned long long)in.delta_ppm) * total) /
                                    ((unsigned long long)L * 1000000ull));
    }
    __syncthreads();
    cap = sh_ctl[1];
    return sh_ctl[0] != 0;
}

// pf[x] = FLOP of operators 0..x-1 (int64); win[n] = number of feasible first operators of a layer that ends
// with the n-th (1-based); meta[0] = the largest of them (at least 1), meta[1] = work counter, meta[2] = a wait
// has run out.  One block.
__global__ __launch_bounds__(CL_THREADS) void cluster_prefix_kernel(
    const int32_t *__restrict__ flop, int K, int64_t cap, ClusterInputs in, int64_t *__restrict__ ctl,
    int64_t *__restrict__ pf, int32_t *__restrict__ win, int64_t *__restrict__ tot, int32_t *__restrict__ meta)
{
    extern __shared__ int64_t sh[];                  // [K + 1] prefix sums
    __shared__ int64_t part[CL_THREADS / WAVE];
    __shared__ int sh_max;
    // Device-resident inputs (ctl) are checked here.  Those that are refused have no feasible first
    // operator anywhere: with a negative figure a row value could be any number, NOT_YET among them.
    const bool refused = ctl && cluster_check(flop, K, in, ctl, cap);
    const int t = threadIdx.x;
    const int per = (K + CL_THREADS - 1) / CL_THREADS;
    const int lo = min(K, t * per), hi = min(K, lo + per);
    int64_t s = 0;
    for (int x = lo; x < hi; ++x) s += flop[x];
    int64_t upto = s;                                // of the wave's lanes up to this one
    for (int off = 1; off < WAVE; off <<= 1) {
        const int64_t o = __shfl_up(upto, off, WAVE);
        if ((t & (WAVE - 1)) >= off) upto += o;
    }
    if ((t & (WAVE - 1)) == WAVE - 1) part[t / WAVE] = upto;
    if (t == 0) { sh_max = 1; sh[0] = 0; }
    __syncthreads();
    int64_t run = upto - s;
    for (int w = 0; w < t / WAVE; ++w) run += part[w];
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

// The band, empty, and the rows of the first launch: row 0 is the empty prefix alone, the others are not there yet
__global__ void cluster_clear_kernel(int64_t *__restrict__ band, int64_t *__restrict__ G, int64_t *__restrict__ V, int K, int rows,
                                     const int32_t *__restrict__ meta)
{
    const long long n = (long long)meta[0] * K, m = (long long)(rows + 1) * (K + 1);
    const long long stride = (long long)gridDim.x * blockDim.x, x0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    for (long long x = x0; x < n; x += stride) band[x] = 0;
    for (long long x = x0; x < m; x += stride) {
        G[x] = x == 0 ? 0 : x <= K ? INF_I64 : NOT_YET;
        V[x] = x <= K ? 0 : NOT_YET;
    }
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

// Rows of a launch that is not the first: row 0 is the row in front (the empty prefix alone for the first of the exact run, else the
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

// (g, v): smaller is better, component by component.  No branches: a row is a chain of these.
struct Lex { uint64_t g, v; };
__device__ __forceinline__ bool lex_not_above(const Lex &a, const Lex &b)
{
    return (a.g < b.g) | ((a.g == b.g) & (a.v <= b.v));
}
template <int CTRL, bool EXACT>
__device__ __forceinline__ void lex_step(Lex &a)
{
    const Lex o{(uint64_t)dpp_mov64<CTRL>((int64_t)a.g), EXACT ? 0 : (uint64_t)dpp_mov64<CTRL>((int64_t)a.v)};
    const bool take = EXACT ? o.g < a.g : lex_not_above(o, a);
    a.g = take ? o.g : a.g;
    if (!EXACT) a.v = take ? o.v : a.v;
}

__device__ __forceinline__ int64_t row_value(const int64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The value at p once it is there (v: what was there at the first look).  Every wait of a call that has the work memory to itself
// ends by itself (see cluster_rows_kernel); what another call overwrites may never come, so after max_spins further looks, or once
// some wait has run out (*lost), the caller goes on without it and the call reports it.  (A clock in the place of
// the count is 2 % of the whole call.)
__device__ __forceinline__ int64_t await(int64_t v, const int64_t *p, int32_t *lost, unsigned max_spins)
{
    for (unsigned spin = 0; v == NOT_YET; ++spin) {
        if (spin >= max_spins ||
            (spin % 64 == 63 && __hip_atomic_load(lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            __hip_atomic_store(lost, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return INF_I64;
        }
        v = row_value(p);
    }
    return v;
}

// Rows 1..rows of this launch, 56 prefix lengths to a workgroup (24 with wide windows, see launch_cluster): seven waves compute a row while the last one fetches
// what the tiles in front have of it, for the next row, so a row takes what its computation takes (0.6 us) and the way of a value
// from one workgroup to the next (1.8 us) is paid once a tile instead of once a row.  3002 operators, 96
// layers: 185 us (where every wave fetched for itself before it computed: 243); 386 operators, 32 layers: 37 us.  By 120 prefix
// lengths to a workgroup 202 and 44 us, by 24 220 and 53, with 16 lanes each on 60 198 and 53; asking for two rows at a time
// 206 and 45: a value that is asked for too early is asked for twice.
// A tile reads rows of tiles in front of it only, and tiles are handed out in order, so the workgroup
// that a wait is for has always started and waits itself only for tiles further in front: every
// wait ends.  A value is its own signal (NOT_YET until it is there), so no fence is needed.
// EXACT (the variance tie-break over whole clusterings): with G* = G(K, L) in *gstar_p,
//   W(n, r) = min over the feasible i with C(i, n) <= G* of W(i-1, r-1) + FLOP(o_i..o_n)^2, lowest i on ties.
// room: prefix lengths in front and own that LDS has room for
template <bool EXACT, class FORM>
__global__ __launch_bounds__(FORM::THREADS) void cluster_rows_kernel(
    const int64_t *__restrict__ band, const int64_t *__restrict__ pf, const int32_t *__restrict__ win, int K,
    int rows, int64_t *G, int64_t *V, int32_t *__restrict__ arg, int32_t *meta,
    const int64_t *__restrict__ gstar_p, unsigned max_spins, int room)
{
    constexpr int T = FORM::TILE, GL = FORM::LANES, KEEP = FORM::KEEP, NT = FORM::THREADS, NF = FORM::FETCH, ASK = 4;
    extern __shared__ int64_t sh[];
    __shared__ int sh_tile;
    if (threadIdx.x == 0) sh_tile = atomicAdd(&meta[1], 1);
    __syncthreads();
    const int n0 = sh_tile * T;                      // the tile: prefix lengths n0 + 1 .. n0 + T
    if (n0 >= K) return;
    const int g = threadIdx.x % GL, nl = threadIdx.x / GL, lane = threadIdx.x & (WAVE - 1);
    const bool fetches = threadIdx.x >= NT - NF * WAVE;
    const int n = n0 + 1 + nl;
    const int base = max(0, n0 - meta[0] + 1);       // first prefix length that the tile reads
    const int halo = n0 + 1 - base;                  // base .. n0 come from tiles in front
    const size_t ld = (size_t)K + 1;
    // two rows: what is read is the one in front, [halo + T] values of V and of G
    constexpr int ENTRY = EXACT ? 1 : 2;             // V, G
    int64_t *now = sh, *next = sh + ENTRY * room;
    for (int x = threadIdx.x; x < halo + T; x += NT) {
        const int m = min(base + x, K);
        now[ENTRY * x] = V[m];
        if (!EXACT) now[ENTRY * x + 1] = G[m];
    }
    // (no further back than the tile reads, whatever another call may have left in `win`)
    const int width = n <= K && !fetches ? min(win[n], n - base) : 0;
    const int64_t pn = pf[min(n, K)];
    const int64_t gstar = EXACT ? *gstar_p : 0;
    // FLOP(o_i..o_n)^2, i = n - j (a layer's FLOP fits 31 bits)
    auto squared = [&](int j) {
        const uint32_t f = (uint32_t)(pn - pf[n - 1 - j]);
        return (int64_t)((uint64_t)f * f);
    };
    // candidate j = g + u * 8; what is none has an infinite cost (in the exact run FLOP^2, and what costs more than G* is none)
    uint64_t keep_c[KEEP], keep_f[KEEP];
    int keep_x[KEEP], terms = 0;                     // terms: how many u the wave has
#pragma unroll
    for (int u = 0; u < KEEP; ++u) {
        const int j = g + u * GL;
        const int64_t c = j < width ? band[(size_t)j * K + n - 1] : INF_I64;
        const bool none = j >= width || (EXACT && (gstar == INF_I64 || c > gstar));
        keep_c[u] = c;
        keep_f[u] = !none ? (uint64_t)squared(j) : EXACT ? (uint64_t)INF_I64 : 0;
        keep_x[u] = ENTRY * max(n - 1 - j - base, 0);                // prefix length i - 1, i = n - j
        terms += __ballot(j < width) != 0;
    }
    __syncthreads();
    if (fetches) {
        for (int r = 1; r <= rows; ++r) {            // row r of the tiles in front, for row r + 1 (the last row's for nobody)
            for (int x0 = ((int)threadIdx.x - (NT - NF * WAVE)) / WAVE * ASK * WAVE; r < rows && x0 < halo; x0 += NF * ASK * WAVE) {
                int64_t v[ASK], w[ASK];
#pragma unroll
                for (int u = 0; u < ASK; ++u) {
                    if (x0 + u * WAVE >= halo) continue;
                    const size_t at = r * ld + base + min(x0 + u * WAVE + lane, halo - 1);
                    v[u] = row_value(&V[at]);
                    if (!EXACT) w[u] = row_value(&G[at]);
                }
#pragma unroll
                for (int u = 0; u < ASK; ++u) {
                    const int x = x0 + u * WAVE + lane, m = base + x;
                    if (x >= halo) continue;
                    // G(0, r) of a positive number of layers is infinite; nobody owns it
                    if (!EXACT) next[ENTRY * x + 1] = m == 0 ? INF_I64 : await(w[u], &G[r * ld + m], &meta[2], max_spins);
                    next[ENTRY * x] = m == 0 ? (EXACT ? INF_I64 : 0) : await(v[u], &V[r * ld + m], &meta[2], max_spins);
                }
            }
            lds_barrier();
            int64_t *const t = now;
            now = next;
            next = t;
        }
        return;
    }
    for (int r = 1; r <= rows; ++r) {
        // (EXACT: W in g.  Sums of an infinite W and a square stay below 2^64)
        Lex best{(uint64_t)INF_I64, 0};
        int at = 0;                                  // its j + 1; of equals the largest
        auto better = [&](const Lex &cur, int j) {
            const bool take = EXACT ? cur.g <= best.g : lex_not_above(cur, best);
            best.g = take ? cur.g : best.g;
            if (!EXACT) best.v = take ? cur.v : best.v;
            at = take ? j + 1 : at;
        };
        auto larger = [](uint64_t a, uint64_t b) { return a > b ? a : b; };
        auto kept = [&](auto count) {
            constexpr int N = decltype(count)::value;
            uint64_t v[N], gp[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                v[u] = now[keep_x[u]];
                if (!EXACT) gp[u] = now[keep_x[u] + 1];
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                better(EXACT ? Lex{v[u] + keep_f[u], 0} : Lex{larger(gp[u], keep_c[u]), v[u] + keep_f[u]}, g + u * GL);
        };
        if (terms <= 4) kept(std::integral_constant<int, 4>());
        else if (terms <= 8) kept(std::integral_constant<int, 8>());
        else kept(std::integral_constant<int, KEEP>());
        for (int j = g + KEEP * GL; j < width; j += GL) {
            const int x = ENTRY * (n - 1 - j - base);
            const uint64_t c = band[(size_t)j * K + n - 1], ff = squared(j);
            if (EXACT) {
                if (gstar != INF_I64 && c <= (uint64_t)gstar) better(Lex{now[x] + ff, 0}, j);
            } else {
                better(Lex{larger(now[x + 1], c), now[x] + ff}, j);
            }
        }
        const Lex own = best;
        lex_step<0xB1, EXACT>(best);             // the n's lanes: neighbours, pairs, quads, halves of a row of 16
        lex_step<0x4E, EXACT>(best);
        lex_step<0x141, EXACT>(best);
        if (GL == 16) lex_step<0x140, EXACT>(best);
        at = (own.g == best.g) & (EXACT | (own.v == best.v)) ? at : 0;
        at = max(at, dpp_mov<0xB1>(at));
        at = max(at, dpp_mov<0x4E>(at));
        at = max(at, dpp_mov<0x141>(at));
        if (GL == 16) at = max(at, dpp_mov<0x140>(at));
        if (g == 0 && n <= K) {
            const bool none = best.g >= (uint64_t)INF_I64;
            const int64_t G_n = none ? INF_I64 : (int64_t)best.g, V_n = EXACT ? G_n : none ? 0 : (int64_t)best.v;
            if (!EXACT) __hip_atomic_store(&G[r * ld + n], G_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&V[r * ld + n], V_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!EXACT) next[ENTRY * (halo + nl) + 1] = G_n;
            next[ENTRY * (halo + nl)] = V_n;
            arg[(r - 1) * ld + n] = none ? 0 : n - at + 1;
        }
        if (threadIdx.x == 0 && n0 == 0) {       // G(0, r), for the row that the next launch starts from
            if (!EXACT) G[r * ld] = INF_I64;
            V[r * ld] = EXACT ? INF_I64 : 0;
            arg[(r - 1) * ld] = 0;
        }
        lds_barrier();
        int64_t *const t = now;
        now = next;
        next = t;
    }
}

// *keep = G(K, L) of the first run (the second one does not write the G rows)
__global__ void cluster_keep_kernel(const int64_t *__restrict__ G, int64_t *__restrict__ keep) { *keep = *G; }

// out[0] = G(K, L), out[1] = V(K, L); first_op[0..L] by walking arg back (one wave).  out[2] = 0, or ctl[0], the
// status of the argument checks (device-resident inputs), or -4 (ALPA_DP_EHIP) if a wait has run out; "no
// clustering" is reported if that is not 0.
__global__ void cluster_walk_kernel(const int64_t *__restrict__ G, const int64_t *__restrict__ V,
                                    const int32_t *__restrict__ arg, int K, int L,
                                    const int64_t *__restrict__ ctl, const int32_t *__restrict__ meta,
                                    int64_t *__restrict__ out, int32_t *__restrict__ first_op)
{
    // G: G(K, L); V: the sum of squares that goes with it (exact mode: W(K, L))
    const int lane = threadIdx.x;
    const int64_t status = ctl && ctl[0] != 0 ? ctl[0] : meta[2] != 0 ? -4 : 0;
    const int64_t g = status != 0 ? INF_I64 : *G;
    if (lane == 0) {
        out[2] = status;
        out[0] = g;
        out[1] = g == INF_I64 ? 0 : *V;
    }
    if (g == INF_I64) {
        for (int r = lane; r <= L; r += WAVE) first_op[r] = -1;
        return;
    }
    int n = K, r = L;
    if (lane == 0) first_op[L] = K;
    // A layer has at most `width` operators: where they fit a wave, what any of the next three rows can be asked for is
    // loaded along with the present one (96 rows: 21 us, a load a row in turn 23)
    const int width = meta[0];
    const size_t ld = (size_t)K + 1;
    while (r >= 1) {
        // lane l: row r - 1 at n; row r - 2 at n - 1 - l; row r - 3 at n - 2 - l and 64 before; row r - 4 at n - 3 - l ..
        auto at = [&](int row, int x) { return arg[(size_t)max(row, 0) * ld + min(max(x, 0), K)]; };
        const bool ahead = width <= WAVE;
        const int a = at(r - 1, n);
        int b = 0, c[2] = {}, d[3] = {};
        if (ahead) {
            b = at(r - 2, n - 1 - lane);
#pragma unroll
            for (int u = 0; u < 2; ++u) c[u] = at(r - 3, n - 2 - lane - u * WAVE);
#pragma unroll
            for (int u = 0; u < 3; ++u) d[u] = at(r - 4, n - 3 - lane - u * WAVE);
        }
        const int from = n;
        auto step = [&](int i) {                     // (i is in 1..n unless another call wrote here)
            n = min(max(i - 1, 0), K);
            --r;
            if (lane == 0) first_op[r] = n;
        };
        auto pick = [&](const int *v, int count, int x) {      // of lane x & 63 of v[x / 64]
            x = min(max(x, 0), count * WAVE - 1);
            int i = 0;
            for (int u = 0; u < count; ++u) i = x / WAVE == u ? __builtin_amdgcn_readlane(v[u], x % WAVE) : i;
            return i;
        };
        step(__builtin_amdgcn_readfirstlane(a));
        if (!ahead) continue;
        if (r >= 1) step(pick(&b, 1, from - 1 - n));
        if (r >= 1) step(pick(c, 2, from - 2 - n));
        if (r >= 1) step(pick(d, 3, from - 3 - n));
    }
}

template <bool EXACT, class FORM>
static hipError_t launch_rows_as(hipStream_t st, const ClusterWork &w, int K, int rows, int width, int32_t *arg,
                                 unsigned max_spins)
{
    constexpr int T = FORM::TILE;
    const auto kernel = cluster_rows_kernel<EXACT, FORM>;
    const int room = std::min(width, K) + T + 1;
    const size_t lds = (size_t)(EXACT ? 2 : 4) * room * sizeof(int64_t);   // (133 KB at most)
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((K + T - 1) / T), dim3(FORM::THREADS), lds, st, w.band,
                       w.pf, w.win, K, rows, w.G, w.V, arg, w.meta, w.keep, max_spins, room);
    return hipGetLastError();
}

template <bool EXACT>
static hipError_t launch_rows(hipStream_t st, const ClusterWork &w, int K, int rows, int width, bool wide, int32_t *arg,
                              unsigned max_spins)
{
    if (wide) return launch_rows_as<EXACT, RowForm<16, 512, 2>>(st, w, K, rows, width, arg, max_spins);
    return launch_rows_as<EXACT, RowForm<8, 512, 1>>(st, w, K, rows, width, arg, max_spins);
}

template <bool EXACT>
static hipError_t launch_run(hipStream_t st, const ClusterWork &w, int K, int L, int width, bool wide, int32_t *arg,
                             unsigned max_spins)
{
    const size_t ld = (size_t)K + 1;
    int done = 0, last = 0;
    while (done < L) {
        const int rows = std::min(ROWS_PER_LAUNCH, L - done);
        if (EXACT || done > 0)
            hipLaunchKernelGGL(cluster_begin_rows_kernel, dim3((K + 64) / 64), dim3(64), 0, st, w.G, w.V, K, rows,
                               done == 0 ? 1 : 0, EXACT ? 1 : 0, last, w.meta);
        const hipError_t e = launch_rows<EXACT>(st, w, K, rows, width, wide, arg + done * ld, max_spins);
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
    hipLaunchKernelGGL(cluster_prefix_kernel, dim3(1), dim3(CL_THREADS), ((size_t)K + 1) * 8, st, flop, K, cap,
                       ClusterInputs{src, dst, nbytes, E, L, delta_ppm}, ctl, w.pf, w.win, w.tot, w.meta);
    const int rows = std::min(L, ROWS_PER_LAUNCH);
    const long long cells = std::max((long long)width * K, (rows + 1ll) * (K + 1));
    hipLaunchKernelGGL(cluster_clear_kernel, dim3((unsigned)std::min<long long>((cells + 1023) / 1024, 1024)),
                       dim3(256), 0, st, w.band, w.G, w.V, K, rows, w.meta);
    if (E > 0)
        hipLaunchKernelGGL(cluster_edges_kernel, dim3((E + 255) / 256), dim3(256), 0, st, src, dst,
                           nbytes, E, K, w.band, w.tot, w.meta);
    hipLaunchKernelGGL(cluster_band_in_kernel, dim3((K + 63) / 64), dim3(64), 0, st, w.band, w.tot, K, w.meta);
    hipLaunchKernelGGL(cluster_band_sum_kernel, dim3((K + 63) / 64), dim3(64), 0, st, w.band, K, w.meta);
    // Windows of more than 128 operators: what eight lanes do not keep in registers they read from memory in every row.  Sixteen lanes and
    // two waves that fetch (device time, us, cell by cell and exact, 8 lanes / 16: 3590 operators, windows of 100
    // 273 and 403 / 285 and 416; 130 276 and 411 / 270 and 399; 200 300 and 499 / 215 and 315; 600 321 and 509 / 238 and 354; 1200 479 and 776 /
    // 328 and 477; 962 operators, 200 113 and 168 / 90 and 124).  Where the width is not known (ctl) it is the narrow form: at most 512 operators, windows of 25
    // 77 / 87, of 200 84 / 73.
    const bool wide = !ctl && width > 128;
    hipError_t e = launch_run<false>(st, w, K, L, width, wide, w.arg, max_spins);
    if (e != hipSuccess) return e;
    const size_t ld = (size_t)K + 1;
    const size_t end = (size_t)((L - 1) % ROWS_PER_LAUNCH + 1) * ld + K;   // (K, L) in the last launch's rows
    if (exact) {
        hipLaunchKernelGGL(cluster_keep_kernel, dim3(1), dim3(1), 0, st, w.G + end, w.keep);
        e = launch_run<true>(st, w, K, L, width, wide, w.arg, max_spins);
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
