// Front costs of a table in LDS (kernels_front.hip, kernels_sparse.hip; gfx950 only).
#pragma once
#include "internal.hpp"

#include <type_traits>

namespace alpa {

typedef int32_t front_v4 __attribute__((ext_vector_type(4)));

constexpr int FRONT_BIG = 1 << 20;             // more devices than there are
constexpr int FRONT_WAVES = 16;                // of a workgroup that finds front costs

__host__ __device__ constexpr int front_blocks(int K) { return (K + 7) / 8; }
__host__ __device__ constexpr int front_groups(int S) { return (S + 7) / 8; }
__host__ __device__ constexpr int front_padded(int S) { return (S + 15) / 16 * 16; }
// A unit: the stages that begin behind row b of P (with layer b) and end in a block of eight rows 8 J + 1 .. 8 J + 8, on eight
// shapes; 64 int32, entry (row & 7, shape & 1) of batch (shape >> 1) & 3 at 4 * entry + batch, +infinity where
// there is no such stage.  Of block J there are units for b = 0 .. 8 J + 7, each of front_groups(S).
__host__ __device__ constexpr int front_units_before(int J) { return 4 * J * (J + 1); }
__host__ __device__ constexpr int front_units(int K, int S) { return front_units_before(front_blocks(K)) * front_groups(S); }

// ---- P in LDS
//
// Row k at k * R, R = D + 2: +infinity, then P(k, 0), P(k, 1), .. P(k, D).  Lanes are device counts; a lane whose count a
// shape exceeds reads the +infinity in front.
struct FrontLds {
    int32_t *P, *tiles, *done;
    int ints;
};
__host__ __device__ __forceinline__ FrontLds front_lds(int32_t *lds, int K, int D, int NG, int W)
{
    FrontLds l;
    int at = 0;
    auto take = [&](int n) { int32_t *p = lds + at; at += (n + 3) & ~3; return p; };
    l.P = take((K + 1) * (D + 2) + 64 * W);    // (lanes beyond D read up to so far behind a row)
    l.tiles = take(2 * 7 * NG * 64);
    l.done = take(W);
    l.ints = at;
    return l;
}

// entry N of the row's 16
template <int N>
__device__ __forceinline__ int32_t front_entry(int32_t t)
{
    return __builtin_amdgcn_update_dpp(0, t, 0x150 + N, 0xf, 0xf, true);
}

// Stages behind one row of P into rows LO .. HI of a block: t are those on 2 N shapes, f the row's cells for each of them.
// (The opaque statements keep the broadcasts with the sums that they are folded into: taken apart they
// are moves, and more registers than there are.)
template <int LO, int HI, int N, bool MAXIMUM>
__device__ __forceinline__ void front_update(int32_t (&acc)[8], int32_t *t, int32_t *f)
{
    auto term = [](int32_t x, int32_t y) { return MAXIMUM ? max(x, y) : x + y; };
#pragma unroll
    for (int x = 0; x < N; ++x) asm volatile("" : "+v"(t[x]), "+v"(f[2 * x]), "+v"(f[2 * x + 1]));
    auto row = [&](auto U) {
        constexpr int u = decltype(U)::value;
        if (u < LO || u > HI) return;
        int32_t s[2 * N];
#pragma unroll
        for (int x = 0; x < N; ++x) {
            s[2 * x] = term(front_entry<u>(t[x]), f[2 * x]);
            s[2 * x + 1] = term(front_entry<u + 8>(t[x]), f[2 * x + 1]);
        }
        if (N == 4) acc[u] = min(min(min(min(s[0], s[1]), s[2]), min(min(s[3], s[4 % (2 * N)]), s[5 % (2 * N)])), min(min(s[6 % (2 * N)], s[7 % (2 * N)]), acc[u]));
        else acc[u] = min(min(min(s[0], s[1]), s[2]), min(s[3], acc[u]));
    };
    row(std::integral_constant<int, 0>{}); row(std::integral_constant<int, 1>{});
    row(std::integral_constant<int, 2>{}); row(std::integral_constant<int, 3>{});
    row(std::integral_constant<int, 4>{}); row(std::integral_constant<int, 5>{});
    row(std::integral_constant<int, 6>{}); row(std::integral_constant<int, 7>{});
#pragma unroll
    for (int u = LO; u <= HI; ++u) asm volatile("" : "+v"(acc[u]));
}

// All of P under the filter `c`, by NW waves, for up to 64 W devices.  In blocks of eight rows: a wave for each window of 64 device
// counts takes the stages inside the block (`triangle`), row by row, while the others take the stages that end in the
// next block (`far`), those that begin inside the present one as its rows come (done: the last row that a window has; a wait
// is for a wave of the same workgroup that never waits for the waiting one).  NH: halves of groups, four shapes each (0: any
// number).  MAXIMUM: the largest stage instead of the sum.  Ends with a barrier.
// Bound by what a wave can issue: a row of the triangle is some 110 instructions of one wave at 5 to 7 clocks each (64
// layers on 8 x 8: 850 clocks a row; 1970 with a branch for each two shapes).
template <int W, int NW, int NH, bool MAXIMUM>
__device__ __forceinline__ void front_costs(const FrontTable &ft, int K, int D, int S, int32_t c, const FrontLds &l)
{
    constexpr int NO = (NW - W) / W, nt = NW * WAVE, NGT = (NH + 1) / 2;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NG = NGT ? NGT : ft.NG, NB = front_blocks(K), R = D + 2, tile_ints = 7 * NG * 64;
    const int size4 = lane < S ? 4 * ft.sizes[lane] : 4 * FRONT_BIG;
    const uint32_t inv_ng = 65536 / NG + 1;        // x / NG for x < 8192
    const bool edge = wid < W;                     // takes the triangles
    const int v = edge ? wid : (wid - W) % W, io = (wid - W) / W;
    const int d = WAVE * v + lane + 1;
    const char *const Pb = (const char *)l.P;
    int32_t *const mine = l.P + 1 + min(d, D);     // the lane's cell of row 0 (lanes beyond D: not to be written)
    // bytes from a row's +infinity to the cell that a shape takes for the lane
    int off[NGT ? NGT : 1][8];
    auto offset = [&](int q) { return max(4 * (d + 1) - __builtin_amdgcn_readlane(size4, q), 0); };
    if (NGT) {
#pragma unroll
        for (int q = 0; q < 8 * NGT; ++q) off[q >> 3][q & 7] = offset(q);
    }
    auto cells = [&](int32_t (&f)[8], int g, int half, int row4) {     // (asks for those of half a group)
        asm volatile("" : "+s"(row4));             // (or a sum for each row and shape of a block is kept, in more registers than there are)
        auto read = [&](const int *o) {
#pragma unroll
            for (int x = 0; x < 4; ++x) f[4 * half + x] = *(const int32_t *)(Pb + (o[x] + row4));
        };
        if (NGT == 1) read(off[0] + 4 * half);
        else if (NGT == 2) {
            if (g == 0) read(off[0] + 4 * half);
            else read(off[NGT ? NGT - 1 : 0] + 4 * half);
        } else {
            int o[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = offset(8 * g + 4 * half + x);
            read(o);
        }
    };
    int32_t ahead = 0;                             // smallest entries of the next 64 units
    auto minima = [&](int T, int x) {
        const int n = T < NB ? (8 * T + 1) * NG : 0;
        return x < n ? ft.unit_min[front_units_before(T) * NG + x] : DEV_INF;
    };
    if (!edge) ahead = minima(0, lane);
    for (int x = tid; x < (K + 1) * R + 64 * W; x += nt) l.P[x] = x == 1 ? 0 : DEV_INF;
    if (tid < W) l.done[tid] = 0;
    lds_barrier();
    auto wait_for = [&](int b, int upto) {         // row b in windows 0 .. upto
        for (int w = 0; w <= upto; ++w)
            while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&l.done[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < b)
                __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    auto triangle = [&](int J) {
        int32_t acc[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[r] = 8 * J + 1 + r <= K ? mine[(8 * J + 1 + r) * R] : DEV_INF;
        const front_v4 *tile = (const front_v4 *)(l.tiles + (J & 1) * tile_ints) + (lane & 15);
        // row r of the block is there: into LDS
        auto put = [&](int r, int32_t value) {
            const int k = 8 * J + 1 + r;
            int at = k * R;
            asm volatile("" : "+s"(at));
            if (d <= D) mine[at] = value;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
            __hip_atomic_store(&l.done[v], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        };
        put(0, acc[0]);
        if (NH != 0 && W == 1) {
            // the next row first, then its cells are asked for while the present one goes into the others
            constexpr int N = NGT ? NGT : 1;
            int32_t f[2][N][8];
            front_v4 t[2][N];
#pragma unroll
            for (int g = 0; g < N; ++g) {
                t[0][g] = tile[g * 16];
                cells(f[0][g], g, 0, 4 * (8 * J + 1) * R);
                if (2 * g + 1 < NH) cells(f[0][g], g, 1, 4 * (8 * J + 1) * R);
            }
            auto row = [&](auto R_T) {
                constexpr int r = decltype(R_T)::value, now = r & 1, then = now ^ 1;
                const int k = 8 * J + 1 + r;
                if (k >= K) return;
                int32_t tv[N][4];
#pragma unroll
                for (int g = 0; g < N; ++g) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) tv[g][x] = t[now][g][x];
                    if (r < 6) t[then][g] = tile[((r + 1) * NG + g) * 16];
                }
                auto into = [&](auto LO, auto HI) {
                    constexpr int lo = decltype(LO)::value, hi = decltype(HI)::value;
                    front_update<lo, hi, NH == 1 ? 2 : 4, MAXIMUM>(acc, tv[0], f[now][0]);
                    if (N > 1) front_update<lo, hi, NH == 3 ? 2 : 4, MAXIMUM>(acc, tv[N - 1], f[now][N - 1]);
                };
                into(std::integral_constant<int, r + 1>{}, std::integral_constant<int, r + 1>{});
                put(r + 1, acc[r + 1]);
                if (r < 6) {
#pragma unroll
                    for (int g = 0; g < N; ++g) {
                        cells(f[then][g], g, 0, 4 * (k + 1) * R);
                        if (2 * g + 1 < NH) cells(f[then][g], g, 1, 4 * (k + 1) * R);
                    }
                    into(std::integral_constant<int, r < 6 ? r + 2 : 7>{}, std::integral_constant<int, 7>{});
                }
            };
            row(std::integral_constant<int, 0>{}); row(std::integral_constant<int, 1>{});
            row(std::integral_constant<int, 2>{}); row(std::integral_constant<int, 3>{});
            row(std::integral_constant<int, 4>{}); row(std::integral_constant<int, 5>{});
            row(std::integral_constant<int, 6>{});
            return;
        }
        auto row = [&](auto R_T) {
            constexpr int r = decltype(R_T)::value;
            const int k = 8 * J + 1 + r;
            if (k >= K) return;
            front_v4 t = tile[r * NG * 16];
            if (W > 1 && v > 0) wait_for(k, v - 1);
            for (int g = 0; g < NG; ++g) {
                front_v4 now = t;
                if (g + 1 < NG) t = tile[(r * NG + g + 1) * 16];
                int32_t f[8], tv[4];
                cells(f, g, 0, 4 * k * R);
                cells(f, g, 1, 4 * k * R);
#pragma unroll
                for (int x = 0; x < 4; ++x) tv[x] = now[x];
                front_update<r + 1, 7, 4, MAXIMUM>(acc, tv, f);
            }
            put(r + 1, acc[r + 1]);
        };
        row(std::integral_constant<int, 0>{}); row(std::integral_constant<int, 1>{});
        row(std::integral_constant<int, 2>{}); row(std::integral_constant<int, 3>{});
        row(std::integral_constant<int, 4>{}); row(std::integral_constant<int, 5>{});
        row(std::integral_constant<int, 6>{});
    };
    // stages into block T from the rows in front of it
    auto far = [&](int T) {
        constexpr int threads = nt - W * WAVE, AHEAD = 4;
        // the stages inside block T that pass, for its triangle: read now, in LDS at the end
        const int4 *const from = (const int4 *)(ft.units + (size_t)(front_units_before(T) + 8 * T + 1) * NG * 64);
        int4 *const tile = (int4 *)(l.tiles + (T & 1) * tile_ints);
        const int x0 = tid - W * WAVE, tile4 = tile_ints / 4;
        const int4 copy = from[min(x0, tile4 - 1)];
        const int n_units = (8 * T + 1) * NG;
        const front_v4 *const units = (const front_v4 *)(ft.units + (size_t)front_units_before(T) * NG * 64) + (lane & 15);
        int32_t acc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = DEV_INF;
        int chunk = -WAVE, turn = io;
        uint64_t left = 0;                         // of the chunk of 64 units: those with a term that nobody has taken
        auto next = [&]() {                        // the next of this wave's (-1: none); source rows ascend
            for (;;) {
                while (left == 0) {
                    chunk += WAVE;
                    if (chunk >= n_units) return -1;
                    left = __ballot(ahead <= c);
                    ahead = minima(T, chunk + WAVE + lane);
                }
                const int bit = __ffsll((unsigned long long)left) - 1;
                left &= left - 1;
                if (turn == 0) {
                    turn = NO - 1;
                    return chunk + bit;
                }
                --turn;
            }
        };
        int u[AHEAD];
        front_v4 t[AHEAD];
        int32_t f[2][8], tv[2][4];
        bool some[2][2];                           // has a half of the group a term?
        const int close = (8 * (T - 1) + 1) * NG;  // from here on units begin behind rows of the present block
        auto ask = [&](int x, const front_v4 &t, int32_t (&cell)[8], int32_t (&tv)[4], bool (&some)[2]) {
            const int b = (int)((uint32_t)x * inv_ng >> 16), g = x - b * NG;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                some[h] = __ballot(min(t[2 * h], t[2 * h + 1]) <= c) != 0;
                tv[2 * h] = t[2 * h] <= c ? t[2 * h] : DEV_INF;
                tv[2 * h + 1] = t[2 * h + 1] <= c ? t[2 * h + 1] : DEV_INF;
            }
            if (x >= close) wait_for(b, v);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (some[h]) cells(cell, g, h, 4 * b * R);
        };
#pragma unroll
        for (int x = 0; x < AHEAD; ++x) {
            u[x] = next();
            t[x] = units[max(u[x], 0) * 16];
        }
        const bool any = u[0] >= 0;
        if (any) ask(u[0], t[0], f[0], tv[0], some[0]);
        for (bool more = any; more;) {
#pragma unroll
            for (int x = 0; x < AHEAD; ++x) {
                const int y = x & 1, z = (x + 1) & 3, then = u[z];
                if (then >= 0 && then < close) ask(then, t[z], f[1 - y], tv[1 - y], some[1 - y]);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (some[y][h]) front_update<0, 7, 2, MAXIMUM>(acc, tv[y] + 2 * h, f[y] + 4 * h);
                u[x] = next();
                t[x] = units[max(u[x], 0) * 16];
                if (then < 0) { more = false; break; }
                if (then >= close) ask(then, t[z], f[1 - y], tv[1 - y], some[1 - y]);
            }
        }
        ahead = minima(T + 1, lane);
        if (any && d <= D) {
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (8 * T + 1 + x <= K) atomicMin(&mine[(8 * T + 1 + x) * R], acc[x]);
        }
        auto passing = [&](int4 x) {
            return make_int4(x.x <= c ? x.x : DEV_INF, x.y <= c ? x.y : DEV_INF, x.z <= c ? x.z : DEV_INF, x.w <= c ? x.w : DEV_INF);
        };
        if (x0 < tile4) tile[x0] = passing(copy);
        for (int x = x0 + threads; x < tile4; x += threads) tile[x] = passing(from[x]);
    };
    // (a loop for each, with as many barriers: what one keeps in registers is nothing to the other)
    if (edge) {
        __builtin_amdgcn_s_setprio(3);             // (what all others wait for)
        lds_barrier();
        for (int J = 0; J < NB; ++J) {
            triangle(J);
            lds_barrier();
        }
        __builtin_amdgcn_s_setprio(0);
    } else {
        for (int T = 0; T < NB; ++T) {
            far(T);
            lds_barrier();
        }
        lds_barrier();
    }
}

// A plan that reaches P(K, D), walked from its last stage on, with stages that have their least latency there where there is a
// choice, and the t_intra it really has (how many stages lie behind each is known now): plan[0] = their sum, plan[1] = the largest; +infinity where a stage has no entry.
__device__ __forceinline__ void front_plan(const FrontTable &ft, const int32_t *__restrict__ table, const BandShapes &bs, int K, int D,
                                           int32_t c, const int32_t *P, int32_t *plan)
{
    __shared__ int sh_term[2], sh_sum, sh_largest;
    __shared__ int sh_stage[256];                  // 64 (first layer, last) + shape of each
    const int S = bs.S, SP = front_padded(S);
    const int32_t *const sizes = bs.sizes;
    const int R = D + 2, tid = threadIdx.x;
    if (tid < 2) sh_term[tid] = INT32_MAX;
    if (tid == 2) sh_sum = 0;
    if (tid == 3) sh_largest = 0;
    lds_barrier();
    int k = K, d = D, n = 0;
    bool found = P[K * R + 1 + D] < DEV_INF;
    while (found && k > 0) {                       // (uniform: every thread walks the same plan)
        const int32_t want = P[k * R + 1 + d];
        int at = INT32_MAX;
        for (int b = tid >> 4; b < k; b += blockDim.x / 16)
            for (int q = tid & 15; q < S; q += 16) {
                const uint32_t e = (uint32_t)((b * K + k - 1) * SP + q);
                const int32_t t = ft.least[e];
                if (t <= c && t + P[b * R + 1 + max(d - sizes[q], -1)] == want) at = min(at, (ft.run[e] > n ? 0 : 1 << 15) + b * 64 + q);
            }
        if (at != INT32_MAX) atomicMin(&sh_term[n & 1], at);
        lds_barrier();
        const int x = __builtin_amdgcn_readfirstlane(sh_term[n & 1]);
        found = x != INT32_MAX;                    // (there is a term)
        if (!found) break;
        const int b = (x & 0x7fff) >> 6, q = x & 63;
        if (tid == 0) {
            sh_term[~n & 1] = INT32_MAX;           // (last read a barrier ago)
            sh_stage[n] = (b * K + k - 1) * 64 + q;
        }
        lds_barrier();
        ++n;
        k = b;
        d -= sizes[q];
    }
    if (tid < n) {
        const int ki = sh_stage[tid] >> 6;
        const int32_t t = band_smallest(table + ((size_t)tid * K * K + ki) * bs.S_table, bs, sh_stage[tid] & 63);
        atomicMax(&sh_largest, t);
        atomicAdd(&sh_sum, t == INF_I32 ? 0 : t);
    }
    lds_barrier();
    if (tid == 0) {
        const bool whole = found && sh_largest != INF_I32;
        plan[0] = whole ? sh_sum : DEV_INF;
        plan[1] = whole ? sh_largest : DEV_INF;
    }
}

// the latency of a plan of one stage (+infinity if there is none)
__device__ __forceinline__ int32_t front_single(const int32_t *__restrict__ table, const BandShapes &bs, int K, int D)
{
    int32_t t = DEV_INF - 1;
    for (int q = 0; q < bs.S; ++q)
        if (bs.sizes[q] == D) t = min(t, band_smallest(table + (size_t)(K - 1) * bs.S_table, bs, q));
    return t;
}

}  // namespace alpa
