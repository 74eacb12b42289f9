// Recurrence kernel (Eq. 3): one workgroup of sixteen waves per t_max candidate, t_intra in bands.
//
// Mapping.  Lanes are device counts, and the first layers k are cut into blocks of 8.  A batch is 16 table
// entries of one submesh shape: the block's first layers against two neighbouring stage LENGTHS (stages k .. k + len - 1),
//     acc[k] = min(acc[k], t[k][len] + F(s-1, k + len, d - a), t[k][len + 1] + F(s-1, k + len + 1, d - a)),
// 16 additions and 8 three-operand minima for 16 cell-updates per lane.  What a filter t_intra <= t_max
// leaves of a table is a band along the diagonal (a longer stage takes longer), so batches by length are full
// where batches by last layer are triangles: with t_max at the low end, where most layers are run, a third of
// the batches (64 layers on 8 x 8: 74 instead of 229 a layer), a quarter less at the high end.
// The operands of neighbouring lengths are the same F rows shifted by one: a unit of four batches (eight
// lengths) reads 15 rows of F for its 64 row-updates of two columns.
//
// t_intra is the same for all lanes of a row of 16: the row loads a unit's 64 entries as four registers (lane l
// holds entry l of each batch, one 16-byte load a lane), and the addition takes its operand from there by a row
// broadcast (DPP row_newbcast), at the full issue rate.  The filter is one compare and one select per batch.
// A shape of a devices has cells only for d >= a + s - 1; where those fit in 32 (16) device counts, two
// (four) neighbouring blocks go through one unit, each in its own half (quarter) of the wave.
//
// F(s-1) and F(s) are buffers of rows F(., first layer, 1..D) in LDS, RS int32 a row and 16 more behind every
// eighth (so that the blocks of one unit lie in different banks); lanes with d - a <= 0 read from a block
// of +infinity behind the buffers.  Three buffers where they fit (the third is cleared while the layer is computed, so
// a layer has one barrier), else two.  Partial minima meet there (ds_min).
//
// Work of a layer: the segments (window of 64 device counts, block group, shape) with an entry for the
// candidate, each of so many batches, dealt to the waves in contiguous shares of equal weight (a unit weighs one more than
// its batches).  The lists are made for several layers ahead, a wave per layer, so that loads of t_intra run
// UNITS_AHEAD units ahead, across segments and layers.
//
// What bounds a round is the slowest candidate's chain of layers (list, shares, units, barrier: 5 to 8 thousand clocks a
// layer at 64 layers on 8 x 8), so what helps is fewer batches and fewer layers.  A whole solve, t_intra by last layer and a
// bound on the sum alone against this (us): 64 layers on 8 x 8, T* of 4096 candidates 1022 and 419; the plan alone out of
// every distinct value 754 and 195; 128 layers, 1024 candidates 2267 and 1059; 64 layers on 16 x 8, 1024: 1060 and 386;
// 48 on 32 x 8, 64 candidates 1186 and 569.
#include "bounds.hpp"

#include <type_traits>

namespace alpa {

constexpr int BAND_TILE = 256;               // int32 per tile: four blocks of 64 (16 entries x 4 batches)
constexpr int BAND_ENDS = 16;
constexpr int BAND_MAX_CELLS = 16384;        // of a layer
constexpr int UNITS_AHEAD = 2;
constexpr int BAND_INF_ROWS = 15;            // rows of the block of +infinity
constexpr int BAND_WAVES = 16;               // per candidate, four per SIMD (eight and four a candidate were slower)
constexpr int BAND_MAX_K = 248;              // (a segment's batches fit seven bits)

__host__ __device__ constexpr int band_blocks(int K) { return (K + 7) / 8; }
// first cell of an F row, and the int32 of a buffer of K + 1 rows (a multiple of four)
__host__ __device__ constexpr int band_row(int r, int RS) { return r * RS + (r >> 3) * 16; }
__host__ __device__ constexpr int band_buffer_ints(int K, int RS) { return band_row(K, RS) + RS; }
// tiles in front of group g (of four blocks): unit u of block hb is there for hb + u < NHB
__host__ __device__ constexpr int band_tiles_before(int NHB, int g) { return g * NHB - 2 * g * (g - 1); }
__host__ __device__ constexpr int band_tiles(int K)
{
    return band_tiles_before(band_blocks(K), (band_blocks(K) + 3) / 4);
}
// position (in batches) from which `ends` entry j counts
__host__ __device__ constexpr int band_end_pos(int NHB, int j)
{
    constexpr int pos[3][BAND_ENDS] = {{0, 1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28},
                                       {0, 1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48},
                                       {0, 1, 2, 3, 4, 6, 8, 12, 16, 20, 24, 32, 48, 64, 80, 96}};
    return NHB <= 8 ? pos[0][j] : NHB <= 16 ? pos[1][j] : pos[2][j];
}

size_t band_table_ints(int K, int Smax, int S) { return (size_t)Smax * S * band_tiles(K) * BAND_TILE; }
size_t band_ends_ints(int K, int Smax, int S) { return (size_t)Smax * band_blocks(K) * S * BAND_ENDS; }

// int32 of layer 1's records that holds the stage of `len` layers from k on, on shape q
__device__ __forceinline__ size_t band_cell(int P, int NHB, int q, int k, int len)
{
    const int hb = k >> 3, l = len - 1;
    return ((size_t)q * P + band_tiles_before(NHB, hb >> 2) + (l >> 3)) * BAND_TILE + (hb & 3) * 64 +
           ((l & 1) * 8 + (k & 7)) * 4 + ((l >> 1) & 3);
}

// A wave per (s, block, q): the block's units (a lane per entry and batch), and the smallest entry from each of
// eight positions on.  Blocks and units that only fill up a tile are +infinity.  there: see BAND_THERE.
__global__ __launch_bounds__(256) void repack_band_kernel(const int32_t *__restrict__ table, int K, BandShapes b, int n,
                                                          int32_t *__restrict__ recs, int32_t *__restrict__ ends, int32_t *there, int falls)
{
    if (blockIdx.x == 0 && threadIdx.x < 2) there[threadIdx.x] = threadIdx.x ? falls : 0;      // (another table; BAND_FALLS)
    const int S = b.S;
    const int NHB = band_blocks(K), NG = (NHB + 3) / 4, P = band_tiles(K);
    const int lane = threadIdx.x & (WAVE - 1);
    const int n_waves = gridDim.x * (blockDim.x / WAVE);
    for (int e = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6); e < n; e += n_waves) {
        const int q = e % S, hb = (e / S) % (4 * NG), s = e / (S * 4 * NG);
        const int g = hb >> 2;
        int32_t *out = recs + (((size_t)s * S + q) * P + band_tiles_before(NHB, g)) * BAND_TILE + (hb & 3) * 64 + lane;
        const int k = 8 * hb + ((lane >> 2) & 7), first_len = 2 * (lane & 3) + (lane >> 5);   // lane = 4 * entry + batch
        const int32_t *row = table + ((size_t)s * K + k) * K * b.S_table;
        int32_t mn[BAND_ENDS];
#pragma unroll
        for (int j = 0; j < BAND_ENDS; ++j) mn[j] = DEV_INF;
        for (int u = 0; u < NHB - 4 * g; ++u) {
            const int i = k + 8 * u + first_len;
            int32_t v = DEV_INF;
            if (i < K) {                               // (then k < K as well)
                const int32_t t = band_smallest(row + (size_t)i * b.S_table, b, q);
                if (t != INF_I32) v = t;
            }
            out[(size_t)u * BAND_TILE] = v;
#pragma unroll
            for (int j = 0; j < BAND_ENDS; ++j)
                if (4 * u + (lane & 3) >= band_end_pos(NHB, j)) mn[j] = min(mn[j], v);
        }
        if (hb < NHB) {
#pragma unroll
            for (int j = 0; j < BAND_ENDS; ++j) {
                const int32_t m = wave_min_i32(mn[j]);
                if (lane == j) ends[(((size_t)s * NHB + hb) * S + q) * BAND_ENDS + j] = m;
            }
        }
    }
}

hipError_t launch_repack_band(hipStream_t st, const int32_t *table, const Problem &p, const BandShapes &b,
                              int32_t *recs, int32_t *ends, int32_t *bounds, bool falls)
{
    const int K = p.K, Smax = p.Smax;
    const int n = Smax * 4 * ((band_blocks(K) + 3) / 4) * b.S;
    hipLaunchKernelGGL(repack_band_kernel, dim3(std::min((n + 3) / 4, 16384)), dim3(256), 0, st, table, K, b, n,
                       recs, ends, bounds + table_bounds_ints(p) + BAND_THERE, falls ? 1 : 0);
    return hipGetLastError();
}

// entry N of the row's 16
template <int N>
__device__ __forceinline__ int32_t band_entry(int32_t t)
{
    return __builtin_amdgcn_update_dpp(0, t, 0x150 + N, 0xf, 0xf, true);
}

static int band_row_ints(int D);

size_t band_thresholds_ints(int K, int D)
{
    return (size_t)BAND_THRESHOLDS * (K * band_row_ints(D) + 64);
}

// rows U .. U + 3 of batch J of a unit (f[r]: the unit's operand row r)
template <bool MAXIMUM>
__device__ __forceinline__ int32_t band_term(int32_t t, int32_t f) { return MAXIMUM ? max(t, f) : t + f; }
template <int U, int J, bool MAXIMUM>
__device__ __forceinline__ void band_update(int32_t (&acc)[8], int32_t t, const int32_t (&f)[15])
{
    // four rows at a time: eight sums in flight before their minima
    constexpr auto term = band_term<MAXIMUM>;
    const int32_t x0 = term(band_entry<U>(t), f[U + 2 * J]), y0 = term(band_entry<U + 8>(t), f[U + 2 * J + 1]);
    const int32_t x1 = term(band_entry<U + 1>(t), f[U + 2 * J + 1]), y1 = term(band_entry<U + 9>(t), f[U + 2 * J + 2]);
    const int32_t x2 = term(band_entry<U + 2>(t), f[U + 2 * J + 2]), y2 = term(band_entry<U + 10>(t), f[U + 2 * J + 3]);
    const int32_t x3 = term(band_entry<U + 3>(t), f[U + 2 * J + 3]), y3 = term(band_entry<U + 11>(t), f[U + 2 * J + 4]);
    acc[U] = min(acc[U], min(x0, y0));
    acc[U + 1] = min(acc[U + 1], min(x1, y1));
    acc[U + 2] = min(acc[U + 2], min(x2, y2));
    acc[U + 3] = min(acc[U + 3], min(x3, y3));
}

template <int J, bool MAXIMUM>
__device__ __forceinline__ unsigned band_batch(int32_t (&acc)[8], int32_t t, const int32_t (&f)[15], int32_t c)
{
    const bool pass = t <= c;
    if (__ballot(pass) == 0) return 0;
    const int32_t tv = pass ? t : DEV_INF;
    band_update<0, J, MAXIMUM>(acc, tv, f);
    band_update<4, J, MAXIMUM>(acc, tv, f);
    return 16;
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int band_prefix_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // last lane of rows 0, 2 to rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // lane 31 to rows 2, 3
    return v;
}

__device__ __forceinline__ bool band_can_skip(const int64_t *chunk_min, int j, int32_t c, int B, int lane)
{
    const int g = j / PRUNE_CHUNK;
    int64_t m = INF_I64;
    for (int x = lane; x < g; x += WAVE)
        m = min64(m, __atomic_load_n(&chunk_min[x], __ATOMIC_RELAXED));
    m = wave_min_i64(m);
    return m != INF_I64 && (int64_t)B * (int64_t)c >= m;
}

struct BandArgs {
    Problem p;
    BandShape b;
    int n_lo, n_hi;
    const int32_t *recs, *ends, *sizes, *cand, *list, *n_list_p;
    int32_t *ticket;
    unsigned long long *wave_relax;
    int64_t *chunk_min;
    int prune, descending;
    int32_t *Fmin, *Sbest;
    int dummy_idx;
    int32_t *F_all;
    const int32_t *s_top_p, *s_bound;
    const int32_t *thr;      // launch_band_bounds
    int32_t max_finite;
    const int32_t *whole, *n_whole_p;      // see FastArgs
    int32_t *rest, *thin;
    int leave_out;
    const int32_t *B_vals;
    int n_B;
};

// Lists of which much is left (of a list that graphs were to settle it may be all: rounds are planned for graphs then): knots first,
// and then what lies between two that differ, in the same launch (us, later calls, with all of it evaluated and so: 48 layers on 32 x 8, 4096
// candidates 20 160 and 2430; random latencies in order, 24 on 2 x 8, 4096: 287 and 211; 40 on 32 x 8: 1700 and 340).
constexpr int BAND_THIN_KNOTS = 256;
constexpr int BAND_BETWEEN = INT32_MAX - 1;            // (in the place of a candidate) all knots are there
// the launch's: knots that are there, is the rest listed, how many that is, its tickets
enum { THIN_DONE, THIN_READY, THIN_REST, THIN_TICKET };
struct BandThin {
    int n, even, behind, span;                         // entries (0: no such list); knots over the first `span` of them, and behind
    int min_B;
    int pending, rests;                                // a knot is being evaluated; the rest's turn
    int count, leave_out, descending;
    const int32_t *whole, *cand;                       // (arguments would take scalar registers)
    int32_t *Fmin, *rest, *thin, *ticket;
};

__device__ __forceinline__ int band_knot(const BandThin &t, int g)
{
    const bool front = g < t.even;
    const int at = front ? g : g - t.even + 1, m = front ? t.even : t.behind + 1, n = front ? t.span : t.n - t.span + 1;
    return (front ? 0 : t.span - 1) + (m <= 1 ? 0 : (int)((int64_t)at * (n - 1) / (m - 1)));
}

// One wave.  Knots lie evenly up to where F hardly changes (as those of refine_begin_kernel); most: at most so many
__device__ __forceinline__ void band_thin_begin(const BandArgs &a, int n_left, int most, BandThin *sh)
{
    const int lane = threadIdx.x & (WAVE - 1), n = a.whole && n_left > BAND_THIN_FROM ? *a.n_whole_p : 0;
    if (n == 0) {
        if (lane == 0) sh->n = 0;
        return;
    }
    const int32_t stages = a.s_bound[a.p.Smax + 2], flat = a.s_bound[a.p.Smax + 3];
    int lo = 0, hi = n - 1;                            // the first entry not below `flat`
    while (lo < hi) {
        const int step = (hi - lo + WAVE - 1) / WAVE, x = lo + step * (lane + 1) - 1;
        const uint64_t valid = __ballot(x < hi), above = __ballot(x < hi && a.cand[a.whole[min(x, hi)]] >= flat);
        if (above) {
            const int l = __ffsll((unsigned long long)above) - 1;
            hi = lo + step * (l + 1) - 1;
            lo += step * l;
        } else {
            lo += step * __popcll(valid);
        }
    }
    int min_B = a.B_vals ? INT32_MAX : a.p.B;
    for (int x = lane; a.B_vals && x < a.n_B; x += WAVE) min_B = min(min_B, a.B_vals[x]);
    min_B = wave_min_i32(min_B);
    most = min(most, BAND_THIN_KNOTS);
    const int behind = min(n - 1 - lo, stages == -1 ? 1 : most / 4);
    if (lane == 0) *sh = BandThin{n, min(most - behind, lo + 1), behind, lo + 1, min_B, 0, 0, 0, a.leave_out, a.descending, a.whole, a.cand, a.Fmin, a.rest, a.thin, a.ticket};
}

// The complement of the next candidate to evaluate, BAND_BETWEEN for the workgroup whose knot is the last to be there, or INT32_MAX
// (one thread).  All tickets are drawn, so the knots that a wait is for are with workgroups that run and do not wait: every wait ends.
__device__ __forceinline__ int band_thin(BandThin *sh)
{
    const int knots = sh->even + sh->behind;
    auto there = [&] { return __hip_atomic_fetch_add(&sh->thin[THIN_DONE], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == knots - 1; };
    if (!sh->rests) {
        if (sh->pending) {
            sh->pending = 0;
            if (there()) return BAND_BETWEEN;
        }
        for (int g; (g = atomicAdd(sh->ticket, 1)) < knots;) {
            const int j = sh->whole[band_knot(*sh, sh->descending ? knots - 1 - g : g)];
            if (sh->Fmin[j] == F_NOT_YET) {              // (else a graph has settled it)
                sh->pending = 1;
                return ~j;
            }
            if (there()) return BAND_BETWEEN;
        }
        while (__hip_atomic_load(&sh->thin[THIN_READY], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == 0) __builtin_amdgcn_s_sleep(8);
        sh->rests = 1;
    }
    const int x = atomicAdd(&sh->thin[THIN_TICKET], 1), n = __hip_atomic_load(&sh->thin[THIN_REST], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (x >= n) return INT32_MAX;
    return ~__hip_atomic_load(&sh->rest[sh->descending ? n - 1 - x : x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All knots are there: entries between two equal ones get their value, those that cannot get below T at the knot in front for any B (where
// only plans count) and those behind the end of Alg. 1's loop none, and the rest is listed.  knot: room for 2 BAND_THIN_KNOTS.
__device__ __forceinline__ void band_between(BandThin *sh, int32_t *knot)
{
    constexpr int nt = BAND_WAVES * WAVE;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                      // (what is computed of it would be kept in registers through the candidates)
    const int lane = tid & (WAVE - 1), n = sh->n, knots = sh->even + sh->behind;
    int32_t *const F = knot + knots;
    for (int g = tid; g < knots; g += nt) {
        const int x = band_knot(*sh, g);
        knot[g] = x;
        F[g] = __hip_atomic_load(&sh->Fmin[sh->whole[x]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    for (int x0 = 0; x0 < n; x0 += nt) {
        const int x = x0 + tid, j = sh->whole[min(x, n - 1)];
        bool evaluate = false;
        if (x < n - 1 && sh->Fmin[j] == F_NOT_YET) {
            int lo = 0, hi = knots - 1;                // knot[lo] <= x < knot[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (knot[mid] <= x) lo = mid; else hi = mid;
            }
            const int32_t fl = F[lo], fr = F[hi];
            int32_t own = F_NOT_YET;
            if (fl == F_SKIPPED || fl == fr) own = fl;
            else if (sh->leave_out && fl < DEV_INF && fr < DEV_INF &&
                     (int64_t)fr - fl + (sh->min_B - 1) * ((int64_t)sh->cand[j] - sh->cand[sh->whole[knot[lo]]]) >= 0) own = F_LEFT_OUT;
            evaluate = own == F_NOT_YET && knot[lo] != x;
            if (own != F_NOT_YET) sh->Fmin[j] = own;
        }
        const uint64_t lanes = __ballot(evaluate);
        int at = 0;
        if (lanes && lane == 0) at = atomicAdd(&sh->count, __popcll(lanes));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(lanes & ((1ull << lane) - 1));
        if (evaluate) __hip_atomic_store(&sh->rest[at], j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (tid == 0) {
        __hip_atomic_store(&sh->thin[THIN_REST], sh->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&sh->thin[THIN_READY], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();                                   // (F's place is the next candidate's)
}

typedef int32_t band_v4 __attribute__((ext_vector_type(4)));

// RS: int32 per F row (device counts of the size class).  NF: front costs that a thread keeps in registers (0: read
// them in every layer).  DUMP: store every layer to F_all (plan recovery: entry j of the list is candidate j itself,
// and only what the walk back from layer s_top_p[j] can reach is computed).  COUNT: tally the executed updates.
// TABLE: no candidate but the table itself, without a filter, in all its layers; F(s, 1, D) goes to a.Fmin[s - 1]
// (TABLE_MAX: with the largest stage instead of the sum).
enum BandMode { BAND_RUN, BAND_COUNT, BAND_DUMP, BAND_TABLE, BAND_TABLE_MAX };
template <int RS, int NF, BandMode MODE>
__device__ __forceinline__ void band_recurrence(const BandArgs &a)
{
    constexpr bool DUMP = MODE == BAND_DUMP, COUNT = MODE == BAND_COUNT, TABLE = MODE >= BAND_TABLE, MAXIMUM = MODE == BAND_TABLE_MAX;
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];
    __shared__ int32_t sh_tk[1];
    __shared__ int32_t sh_skip[BAND_WAVES];
    constexpr int nw = BAND_WAVES, nt = nw * WAVE;
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = a.p.K, D = a.p.D, S = a.p.S, NHB = band_blocks(a.p.K);
    const int LS = (K + 2) * (D + 1);
    const int BUF = band_buffer_ints(K, RS);
    const int P = band_tiles(K);
    const int NO_CELL = a.b.nbuf * BUF;                                      // block of +infinity
    int2 *const units = (int2 *)(lds + NO_CELL + BAND_INF_ROWS * RS + 16); // [ahead][cap]: see `build_lists`
    int32_t *const n_units = (int32_t *)(units + a.b.ahead * a.b.cap);     // [ahead]
    const int NG = (NHB + 3) >> 2, GS = NG * S;
    uint8_t *const lens = (uint8_t *)(lds + a.b.lens_at);                  // [ahead][group][S][block of the group]
    int32_t *const win_lo = lds + a.b.bounds_at, *const win_hi = win_lo + 32;      // [block] device counts it is computed for
    int32_t *const sh_least = win_hi + 32;                                 // [2]: see `hopeless`
    // work lists: lanes over 2^lg_q >= S shapes and `per` blocks, `chunks` times
    const int lg_q = 32 - __builtin_clz((S - 1) | 1), per = WAVE >> lg_q, nh = (NHB + per - 1) / per, chunks = a.b.W * nh;
    const uint32_t inv_nh = 65536 / nh + 1, inv_chunks = (1u << 20) / chunks + 1;  // x / nh, x / chunks for what is divided here
    const int q_of_lane = lane & ((1 << lg_q) - 1), size_q = a.sizes[min(q_of_lane, S - 1)];
    const int n = TABLE ? 1 : __builtin_amdgcn_readfirstlane(*a.n_list_p);
    if (n <= a.n_lo || n > a.n_hi) return;                                 // the other form's share (whole grid)
    unsigned long long rows_total = 0;
    // A unit of several blocks reads past the last buffer where a block has no such unit: its t_intra are
    // +infinity there, and what they are added to may be any number from 0 to +infinity (so may the work lists).
    for (int x = NO_CELL + tid; x < a.b.lens_at; x += nt) lds[x] = DEV_INF;
    __syncthreads();
    const int32_t least_after_1 = DUMP || TABLE ? 0 : a.s_bound[1];         // of any plan of more than one stage
    const int32_t thr_lo = band_threshold(a.max_finite, min(lane, BAND_THRESHOLDS - 1));
    const int32_t thr_hi = band_threshold(a.max_finite, min(lane + WAVE, BAND_THRESHOLDS - 1));

    // The first candidate goes by the workgroup's number, the others are drawn; of a list of which much is left all are, and given by
    // their complement (what that takes is in LDS: there is no register to spare)
    constexpr bool THINS = !DUMP && !TABLE;
    __shared__ BandThin sh_thin;
    if (THINS) {
        if (wid == 0) band_thin_begin(a, n, NO_CELL / 2, &sh_thin);
        __syncthreads();
    }
    auto next = [&](bool first) {
        while (THINS && __builtin_amdgcn_readfirstlane(sh_thin.n) != 0) {
            int t = tid;
            asm volatile("" : "+v"(t));                // (see draw_ticket)
            if (t == 0) *sh_tk = band_thin(&sh_thin);
            __syncthreads();
            const int x = __builtin_amdgcn_readfirstlane(*sh_tk);
            __syncthreads();
            if (x != BAND_BETWEEN) return x;
            band_between(&sh_thin, lds);
        }
        return TABLE ? (first ? 0 : 1) : first ? (int)blockIdx.x : (int)gridDim.x + draw_ticket(a.ticket, tid, sh_tk);
    };
    for (int tk, turn = 0; (tk = next(turn == 0)) < n; ++turn) {
        const int pos = a.descending ? n - 1 - tk : tk;
        const int j = TABLE ? 0 : DUMP ? pos : tk < 0 ? ~tk : __builtin_amdgcn_readfirstlane(a.list[pos]);
        const int32_t c_given = TABLE ? DEV_INF : __builtin_amdgcn_readfirstlane(a.cand[j]);
        const int32_t c = min(c_given, DEV_INF - 1);   // the sentinel entries pass no candidate
        if (!DUMP && !TABLE && a.prune) {
            sh_skip[wid] = band_can_skip(a.chunk_min, j, c_given, a.p.B, lane) ? 1 : 0;
            __syncthreads();
            const int skip = __builtin_amdgcn_readfirstlane(sh_skip[0]);
            __syncthreads();
            if (skip) {
                a.Fmin[j] = F_SKIPPED;                 // all threads, same value
                a.Sbest[j] = -1;
                continue;
            }
        }
        if (DUMP && a.s_top_p[j] < 1) continue;        // (uniform: there is no plan, or it is known)
        // Plan recovery walks back from F(s*, first layer 1, all devices): only layers up to s* are needed,
        // and of layer s only first layers (0-based) s* - s <= k <= K - s
        const int s_top = DUMP ? min(a.p.Smax, __builtin_amdgcn_readfirstlane(a.s_top_p[j])) : a.p.Smax;
        int32_t *F_out = DUMP ? a.F_all + (size_t)j * (size_t)(a.p.Smax + 1) * LS : nullptr;

        // Work lists of layers s0 .. s0 + ahead - 1.  A unit is two words:
        //   A: log2(blocks) | (batches - 1) << 2 | window << 4 | (256-byte position in the layer's records) << 8 | first block << 24
        //   B: first operand cell, less the shape's size | size << 17 | 1 << 29       (0: no unit)
        int made = 1;                                  // lists are there up to this layer
        auto build_lens = [&](int s0, int ln) {        // batches of each (layer, block, shape)
            if (tid < ln) n_units[tid] = 0;
            for (int x = tid; x < ln * 4 * GS; x += nt) {
                const int l = x / (4 * GS), r = (x - l * 4 * GS) >> 2, g = r / S, hb = 4 * g + (x & 3), s = s0 + l;
                const int4 *e = (const int4 *)(a.ends + (((size_t)(s - 1) * NHB + min(hb, NHB - 1)) * S + (r - g * S)) * BAND_ENDS);
                const int4 e0 = e[0], e1 = e[1], e2 = e[2], e3 = e[3];
                const int v[BAND_ENDS] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w,
                                          e2.x, e2.y, e2.z, e2.w, e3.x, e3.y, e3.z, e3.w};
                int len = 0;
#pragma unroll
                for (int y = 0; y < BAND_ENDS; ++y) {
                    const int to = y + 1 < BAND_ENDS ? band_end_pos(NHB, y + 1) : 128;
                    len = v[y] <= c ? to : len;        // (the entries ascend)
                }
                const int span = K - s - 8 * hb;       // the last layer of a stage is at most K - s
                const bool none = hb >= NHB || span < 0 || (DUMP && 8 * hb + 7 < s_top - s);
                lens[x] = (uint8_t)(none ? 0 : min(len, (span >> 1) + 1));
            }
        };
        auto build_lists = [&](int s0, int ln) {       // (in no order but that of a chunk: 64 pairs of a block and a shape)
            for (int task = wid; task < ln * chunks; task += nw) {
                const int l = (int)((task * inv_chunks) >> 20), ch = task - l * chunks;
                const int w = (int)((ch * inv_nh) >> 16), hb = (ch - w * nh) * per + (lane >> lg_q);
                const int d_min = size_q + s0 + l - 1;     // device counts that leave one to each stage behind
                // device counts that the blocks of the group have for the shape in this window
                const int g = min(hb >> 2, NG - 1);
                const uint32_t len4 = ((const uint32_t *)lens)[l * GS + g * S + min(q_of_lane, S - 1)];
                const int4 lo4 = ((const int4 *)win_lo)[g], hi4 = ((const int4 *)win_hi)[g];
                const int los[4] = {lo4.x, lo4.y, lo4.z, lo4.w}, his[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
                int most = 0, len[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int serves = his[b] - max(los[b], d_min) + 1 - WAVE * w;
                    len[b] = serves > 0 ? (int)((len4 >> (8 * b)) & 255) : 0;
                    most = max(most, len[b] > 0 ? serves : 0);
                }
                const int mode = most > 32 ? 0 : most > 16 ? 1 : 2, step = 1 << mode;
                int nb = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (b >= (hb & 3) && b < (hb & 3) + step) nb = max(nb, len[b]);
                if (q_of_lane >= S || hb >= NHB || (hb & (step - 1)) != 0) nb = 0;
                const int n = (nb + 3) >> 2, upto = band_prefix_sum(n);
                int first = 0;
                if (lane == WAVE - 1) first = atomicAdd(&n_units[l], upto);
                int2 *list = units + l * a.b.cap + __builtin_amdgcn_readlane(first, WAVE - 1) + upto - n;
                int A = mode | (3 << 2) | (w << 4) | (((q_of_lane * P + band_tiles_before(NHB, hb >> 2)) * 4 + (hb & 3)) << 8) | (hb << 24);
                int B = (hb * (8 * RS + 16) + RS - size_q) | (size_q << 17) | (1 << 29);
                for (int u = 1; u <= n; ++u, ++list) {
                    *list = make_int2(u < n ? A : A - ((4 * n - nb) << 2), B);
                    A += 4 << 8;
                    B += 8 * RS + 16;
                }
            }
            made = s0 + ln - 1;
        };
        // least plan of more stages than s0 + l, in lanes 32 + l
        constexpr bool BOUNDED = !DUMP && !TABLE;
        auto bounds_of = [&](int s0) { return BOUNDED ? a.s_bound[min(s0 + (lane & 31), a.p.Smax)] : 0; };
        auto counts_of = [&](int32_t bounds) {
            const int n = n_units[min(lane, a.b.ahead - 1)];
            return BOUNDED && lane >= 32 ? bounds : n;
        };
        const int ln2 = min(a.b.ahead, s_top - 1);
        const int32_t bounds2 = bounds_of(2);
        // what is known of the lowest threshold that is not below the candidate (thresholds descend; the first has no filter)
        const int thr_at = max(0, min((int)(__popcll(__ballot(thr_lo >= c)) + __popcll(__ballot(lane + WAVE < BAND_THRESHOLDS && thr_hi >= c))), BAND_THRESHOLDS) - 1);
        const int32_t *w = a.thr + (size_t)BAND_THRESHOLDS * K * RS + 64 * thr_at;
        if (tid < 64) win_lo[tid] = w[tid];
        if (tid < 2) sh_least[tid] = DEV_INF;
        const int32_t *const fronts = a.thr + (size_t)thr_at * K * RS;
        int32_t front[NF ? NF : 1];                    // front costs of cells tid, tid + nt, ..
        if (!DUMP && !TABLE) {
#pragma unroll
            for (int x = 0; x < NF; ++x) front[x] = fronts[min(tid + x * nt, K * RS - 1)];
        }
        for (int x = 4 * tid; x < NO_CELL; x += 4 * nt) *(int4 *)(lds + x) = make_int4(DEV_INF, DEV_INF, DEV_INF, DEV_INF);
        build_lens(2, ln2);
        __syncthreads();
        // layer 1: the only finite operand is F(0, K+1, 0) = 0, so F(1, k, a) is the stage k .. K - 1 on a devices
        for (int x = tid; x < K * S; x += nt) {
            const int q = x / K, k = x - q * K;
            const int32_t t = a.recs[band_cell(P, NHB, q, k, K - k)];
            if (t <= c) atomicMin(&lds[BUF + band_row(k, RS) + a.sizes[q] - 1], t);
        }
        build_lists(2, ln2);
        __syncthreads();
        int32_t best = DEV_INF, sbest = 0;
        unsigned rows = 0;
        auto clear = [&](int F, int last, int by) {    // rows up to `last`, by the first so many threads
            int4 *p = (int4 *)__builtin_assume_aligned(lds + F, 16);
            const int end = band_row(last + 1, RS) >> 2;
            for (int x = tid; x < end; x += by) p[x] = make_int4(DEV_INF, DEV_INF, DEV_INF, DEV_INF);
        };
        // after layer s: does it end here?  (`least`: of any plan of more stages)
        auto finished = [&](int s, int F, int32_t least) {
            const int32_t f1 = __builtin_amdgcn_readfirstlane(lds[F + D - 1]);     // F(s, first layer, all devices)
            if (f1 < best) { best = f1; sbest = s; }   // lowest s on ties
            if (TABLE && tid == 0) a.Fmin[s - 1] = min(f1, DEV_INF);
            return !DUMP && !TABLE && least >= best;
        };
        // Can no plan that goes on from layer s be below what there is?  (A barrier; uniform.)
        auto hopeless = [&](int s, int F) {
            int32_t m = DEV_INF;
            auto cell = [&](int e, int32_t f) { m = min(m, lds[F + e + e / (8 * RS) * 16] + f); };
            if (NF) {
                // (eight registers: for layers of more than four cells a thread; the first four are at constant distances, which takes no
                // registers for where they are)
                static_assert(nt % (8 * RS) == 0 || 8 * RS % nt == 0);
#pragma unroll
                for (int x = 0; x < NF; ++x) {
                    if (NF == 8 && x < 4) m = min(m, lds[F + tid + (nt > 8 * RS ? tid / (8 * RS) * 16 : 0) + x * nt + x * nt / (8 * RS) * 16] + front[x]);
                    else cell(min(tid + x * nt, K * RS - 1), front[x]);
                }
            } else {
                for (int x = 0; x < K * RS; x += 4 * nt) {
                    int32_t f[4];
#pragma unroll
                    for (int y = 0; y < 4; ++y) f[y] = fronts[min(tid + x + y * nt, K * RS - 1)];
#pragma unroll
                    for (int y = 0; y < 4; ++y) cell(min(tid + x + y * nt, K * RS - 1), f[y]);
                }
            }
            m = wave_min_i32(m);
            if (lane == 0) atomicMin(&sh_least[s & 1], m);
            lds_barrier();
            const bool h = __builtin_amdgcn_readfirstlane(sh_least[s & 1]) >= best;
            if (tid == 0) sh_least[~s & 1] = DEV_INF;  // (for the next layer; last read a barrier ago)
            return h;
        };
        auto dump = [&](int s, int F) {                // (column 0 and what the walk cannot reach stay as they are)
            int32_t *out = F_out + (size_t)s * LS;
            for (int r = max(0, s_top - s) + wid; r <= K - s; r += nw / 2)
                for (int x = lane; x < D; x += WAVE) out[(uint32_t)((r + 1) * (D + 1) + 1 + x)] = lds[F + band_row(r, RS) + x];
        };

        // The wave's units, in order over the layers: a layer's share goes through a ring of UNITS_AHEAD loads in
        // whole rounds, filled up with empty units.  w_A, w_B: up to 64 units of the share, a lane each.
        int w_base = 2;                                // first layer of the lists
        int w_counts = counts_of(bounds2);             // lane l: units of layer w_base + l; and bounds
        int b_base = 2;                                // layer of the first bound
        int w_A = 0, w_B = 0, w_at = 0, w_first = 0, w_end = 0;
        uint32_t w_layer = 0;                          // where the layer's records begin (in bytes)
        const uint32_t lane_16 = (lane & 15) << 4, lane_128 = (lane >> 4) << 7;
        auto fetch = [&](int l) {                      // the next 64 units of the share
            const int x = w_first + lane;
            const int2 u = units[l * a.b.cap + min(x, a.b.cap - 1)];
            w_A = x < w_end ? u.x : 0;
            w_B = x < w_end ? u.y : 0;
            w_at = 0;
        };
        auto enter = [&](int s) {                      // returns the rounds of layer s
            const int l = s - w_base, all = __builtin_amdgcn_readlane(w_counts, l);
            w_first = (all * wid) / nw;
            w_end = (all * (wid + 1)) / nw;
            w_layer = (uint32_t)(s - 1) * (uint32_t)(S * P * BAND_TILE * 4);
            fetch(l);
            return (int)max(1u, (unsigned)(w_end - w_first + UNITS_AHEAD - 1) / (unsigned)UNITS_AHEAD);
        };
        int rA[UNITS_AHEAD], rB[UNITS_AHEAD];
        band_v4 t[UNITS_AHEAD];
        auto load = [&](int x) {
            rA[x] = __builtin_amdgcn_readlane(w_A, w_at + x);
            rB[x] = __builtin_amdgcn_readlane(w_B, w_at + x);
            // lanes of a row of 16 share a block: log2(blocks) 0, 1, 2 puts rows 0..3 at blocks 0000, 0011, 0123
            const uint32_t at = ((lane_128 * (uint32_t)(rA[x] & 3)) & 0x300) + lane_16 + (w_layer + (uint32_t)(rA[x] & 0xffff00));
            t[x] = *(const band_v4 *)((const char *)a.recs + at);
        };

        int Fp = BUF, Fn = a.b.nbuf > 2 ? 2 * BUF : 0, Fc = 0;     // buffers of layers s - 1, s and (to be) s + 1
        bool done = s_top < 1 || finished(1, Fp, least_after_1);
        if (s_top < 2) done = true;
        if (!DUMP && !TABLE && !done && best < DEV_INF) done = hopeless(1, Fp);
        int rounds = 0;                                // of layer s; its first units are in the ring
        if (!done) {
            rounds = enter(2);
#pragma unroll
            for (int x = 0; x < UNITS_AHEAD; ++x) load(x);
        }
        for (int s = 2; !done; ++s) {
            if (s > made) {
                const int ln = min(a.b.ahead, s_top - s + 1);
                int32_t bounds = w_counts;
                if (BOUNDED && s + ln > b_base + 32) {
                    b_base = s;
                    bounds = bounds_of(s);
                }
                build_lens(s, ln);
                lds_barrier();
                build_lists(s, ln);
                lds_barrier();
                w_base = s;
                w_counts = counts_of(bounds);
                rounds = enter(s);
#pragma unroll
                for (int x = 0; x < UNITS_AHEAD; ++x) load(x);
            }
            int rounds_next = 0;
            int key = -1, dl = 0, rp = 0, out = 0;
            int32_t acc[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[u] = DEV_INF;
            auto flush = [&]() {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    atomicMin(&lds[out + u * RS], acc[u]);
                    acc[u] = DEV_INF;
                }
            };
#pragma nounroll
            for (; rounds > 0; --rounds) {
                w_at += UNITS_AHEAD;
                if (rounds == 1) {                     // what is loaded in the last round is the next layer's
                    if (s < made) rounds_next = enter(s + 1);
                    else w_A = w_B = w_at = 0;
                } else if (w_at == WAVE) {
                    w_first += WAVE;
                    fetch(s - w_base);
                }
#pragma unroll
                for (int x = 0; x < UNITS_AHEAD; ++x) {
                    if (rB[x] != 0) {
                        const int A = rA[x], B = rB[x];
                        if ((A & 0xff000033) != key) { // another block group: its own accumulators
                            if (key >= 0) flush();
                            key = A & 0xff000033;
                            const int mode = A & 3, width = WAVE >> mode;
                            const int sub = lane >> (6 - mode), block = min((A >> 24) + sub, NHB - 1);
                            dl = win_hi[block] - WAVE * ((A >> 4) & 3) - width + (lane & (width - 1));     // the lane's device count - 1
                            rp = sub * (8 * RS + 16) + dl;
                            out = dl >= 0 ? Fn + (A >> 24) * (8 * RS + 16) + rp : NO_CELL;
                        }
                        // rows 1 .. 7 of the operand block, and 0 .. 7 of the next
                        const int fa = dl >= ((B >> 17) & 1023) ? Fp + (B & 0x1ffff) + rp : NO_CELL;
                        const int32_t *f0 = lds + fa, *f1 = lds + (fa + 16);
                        const band_v4 tt = t[x];
                        int32_t f[15];
#pragma unroll
                        for (int r = 0; r < 7; ++r) f[r] = f0[r * RS];
                        f[7] = f1[7 * RS];
                        f[8] = f1[8 * RS];
                        if ((A & 12) != 0) {           // more than one batch
#pragma unroll
                            for (int r = 9; r < 15; ++r) f[r] = f1[r * RS];
                        }
                        // (one `if` behind the other: where they nest the accumulators are copied at every join)
                        unsigned did = band_batch<0, MAXIMUM>(acc, tt.x, f, c);
                        if ((A & 12) != 0) did += band_batch<1, MAXIMUM>(acc, tt.y, f, c);
                        if ((A & 8) != 0) did += band_batch<2, MAXIMUM>(acc, tt.z, f, c);
                        if ((A & 8) != 0) did += band_batch<3, MAXIMUM>(acc, tt.w, f, c);
                        if (COUNT) rows += did;
                    }
                    load(x);
                }
            }
            rounds = rounds_next;
            if (key >= 0) flush();
            if (wid < nw / 2) {                        // (the lower waves go first on their SIMD and have time)
                if (a.b.nbuf > 2) clear(Fc, min(K - 1, K - s + 2), nt / 2);    // the next layer's buffer: nobody reads it any more
                if (DUMP) dump(s - 1, Fp);
            }
            lds_barrier();
            done = finished(s, Fn, DUMP || TABLE ? 0 : __builtin_amdgcn_readlane(w_counts, 32 + s - b_base)) || s == s_top;
            if (!DUMP && !TABLE && !done && best < DEV_INF) done = hopeless(s, Fn);
            if (a.b.nbuf > 2) {
                const int f = Fp;
                Fp = Fn; Fn = Fc; Fc = f;
            } else if (!done) {
                clear(Fp, K - s + 1, nt);
                const int f = Fp;
                Fp = Fn; Fn = f;
                lds_barrier();
            } else {
                Fp = Fn;
            }
        }
        if (DUMP && s_top >= 1 && wid < nw / 2) dump(s_top, Fp);
        if (TABLE) return;
        const int slot = wid == 0 ? j : a.dummy_idx;   // wave 0 owns the result
        a.Fmin[slot] = best;                           // all lanes, same value
        a.Sbest[slot] = best >= DEV_INF ? 0 : sbest;
        if (a.prune && best < DEV_INF)                 // uniform
            publish_min(&a.chunk_min[j / PRUNE_CHUNK], (int64_t)best + (int64_t)(a.p.B - 1) * (int64_t)c_given, tid);
        if (COUNT) rows_total += rows;
        __syncthreads();                               // LDS is reused by the next candidate
    }
    if (COUNT) atomicAdd(a.wave_relax, lane == 0 ? rows_total : 0ull);
}

template <int RS, int NF, bool DUMP, bool COUNT>
__global__ __launch_bounds__(WAVE * BAND_WAVES) void recurrence_band_kernel(BandArgs a)
{
    band_recurrence<RS, NF, DUMP ? BAND_DUMP : COUNT ? BAND_COUNT : BAND_RUN>(a);
}

// The bounds of a table that no graphs are made for (sparse_graph_kernel), a workgroup for each threshold.
constexpr int BAND_BOUNDS_THREADS = 512;
__global__ __launch_bounds__(BAND_BOUNDS_THREADS) void band_bounds_kernel(Problem p, int32_t max_finite, const int32_t *__restrict__ table,
                                                                          BandShapes bs, const int32_t *__restrict__ fronts, int RS,
                                                                          const int32_t *__restrict__ totals, int32_t *plans,
                                                                          int32_t *__restrict__ bounds, int once, int32_t *there)
{
    if (once && *there) return;
    band_bounds(p, max_finite, table, bs, fronts, RS, totals, plans, bounds, there, blockIdx.x);
}

// Where the thresholds say little, the recurrence itself without a filter, through all its layers, in two workgroups: one for the
// sum, one for the largest stage.  That takes 0.4 (64 layers on 8 x 8) to 2 ms (48 on 32 x 8), so it is done for a table that is
// solved a second time.  (Random latencies, us, later solves with and without: 64 layers on 8 x 8, 4096 candidates 205 and
// 2309; 48 on 32 x 8, 300 candidates, the plan alone 405 and 1499.)
template <int RS>
__global__ __launch_bounds__(WAVE * BAND_WAVES) void band_exact_bounds_kernel(BandArgs a, const int32_t *__restrict__ totals,
                                                                             const int32_t *__restrict__ plans, int32_t *__restrict__ bounds,
                                                                             int once, int32_t *there)
{
    const int Smax = a.p.Smax, tid = threadIdx.x, half = blockIdx.x == 0 ? 2 : 4;
    if ((once && (*there & half)) || !band_bounds_poor(totals, band_best_plan(plans))) return;
    if (blockIdx.x == 0) {
        band_recurrence<RS, 0, BAND_TABLE>(a);
        __syncthreads();
        // bounds[s]: the least of more than s stages.  From the least of all on F does not change: no stage is larger.
        int32_t m = DEV_INF;
        if (tid <= Smax) {
            for (int x = tid; x < Smax; ++x) m = min(m, a.Fmin[x]);
            bounds[tid] = m;
        }
        if (tid == 0) bounds[Smax + 3] = m;
    } else {
        a.Fmin = a.Sbest;
        band_recurrence<RS, 0, BAND_TABLE_MAX>(a);
        __syncthreads();
        if (tid == 0) {
            int32_t g = DEV_INF, sg = 0;
            for (int x = 0; x < Smax; ++x) {
                const int32_t v = a.Sbest[x];
                if (v < g) { g = v; sg = x + 1; }
            }
            bounds[Smax + 1] = g;
            bounds[Smax + 2] = sg;
        }
    }
    if (tid == 0) atomicOr(there, half);
}

// F rows of the size class that holds D devices (0: none does)
static int band_row_ints(int D) { return D <= 64 ? 64 : D <= 128 ? 128 : D <= 256 ? 256 : 0; }

// How a problem goes through the kernel (nbuf = 0: it does not).  `sizes`: devices of each shape
BandShape band_shape(int K, int D, int S, const int32_t *sizes)
{
    BandShape b{};
    const int RS = band_row_ints(D), NHB = band_blocks(K);
    if (RS == 0 || K > BAND_MAX_K || K * RS > BAND_MAX_CELLS) return b;
    b.W = (D + WAVE - 1) / WAVE;
    // the most units a layer can have: layer 2, every block of every shape to its end
    for (int w = 0; w < b.W; ++w)
        for (int q = 0; q < S; ++q) {
            const int rem = D - WAVE * w - sizes[q];
            const int step = rem > 32 ? 1 : rem > 16 ? 2 : 4;
            for (int hb = 0; rem > 0 && hb < NHB; hb += step) b.cap += NHB - hb;
        }
    b.cap = std::max(b.cap, 1);
    const int most = (160 * 1024 - 256) / 4;           // less the kernel's few static words
    for (int nbuf = 3; nbuf >= 2; --nbuf) {
        const int f = nbuf * band_buffer_ints(K, RS);
        for (int ahead = std::min(16, std::max(1, std::min(K, D) - 1)); ahead >= (nbuf == 3 ? 2 : 1); --ahead) {
            const int lists = f + BAND_INF_ROWS * RS + 16 + ahead * (2 * b.cap + 1);
            // (a unit of four blocks reads up to 38 rows behind row K)
            const int lens = (std::max(lists, f + 38 * RS + 5 * 16) + 3) & ~3;
            const int bounds = (lens + ahead * ((NHB + 3) / 4) * S + 3) & ~3, all = (bounds + 64 + 2 + 3) & ~3;
            if (all <= most) {
                b.nbuf = nbuf;
                b.ahead = ahead;
                b.lens_at = lens;
                b.bounds_at = bounds;
                b.lds_ints = all;
                return b;
            }
        }
    }
    return b;
}

// behind the bounds: BAND_TOTALS (totals, plans)
hipError_t launch_band_bounds(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                              const BandWork &w, int32_t *bounds, bool once)
{
    int32_t *totals = bounds + table_bounds_ints(p), *plans = totals + BAND_THRESHOLDS + 1, *there = totals + BAND_THERE;
    const int32_t *const asked = once ? there : nullptr;
    const int RS = band_row_ints(p.D);
    int32_t *const thr = w.thr;
    hipError_t e = launch_front_thresholds(st, table, b, p, max_finite, w.least, w.front, thr, w.backs, totals, plans,
                                           thr + (size_t)BAND_THRESHOLDS * p.K * RS, w.graph ? graph_used(w.graph, p.K, p.D) : nullptr, asked);
    if (e == hipSuccess && w.graph)
        return launch_sparse_graph(st, table, b, p, max_finite, w.least, w.front, thr, w.backs, totals, plans, totals + BAND_FALLS, w.graph,
                                   bounds, there, once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(band_bounds_kernel, dim3(BAND_THRESHOLDS), dim3(BAND_BOUNDS_THREADS), 0, st, p, max_finite, table, b, thr, RS,
                       totals, plans, bounds, once, there);
    return hipGetLastError();
}

// behind launch_band_bounds of the same table, with the same arrays (`once`: see there)
hipError_t launch_band_exact_bounds(hipStream_t st, const BandShapes &b, const BandShape &shape, const Problem &p, int32_t max_finite,
                                    const int32_t *recs, const int32_t *ends, int32_t *work, const int32_t *thr, int32_t *bounds, bool once)
{
    int32_t *totals = bounds + table_bounds_ints(p), *plans = totals + BAND_THRESHOLDS + 1, *there = totals + BAND_THERE;
    const int RS = band_row_ints(p.D);
    BandArgs a{p, shape, -1, INT32_MAX, recs, ends, b.sizes};
    a.p.S = b.S;
    a.Fmin = work;
    a.Sbest = work + p.Smax;
    a.thr = thr;
    a.max_finite = max_finite;
    const auto kernel = RS == 64 ? band_exact_bounds_kernel<64> : RS == 128 ? band_exact_bounds_kernel<128> : band_exact_bounds_kernel<256>;
    const size_t lds = (size_t)shape.lds_ints * 4;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(2), dim3(WAVE * BAND_WAVES), lds, st, a, totals, plans, bounds, once, there);
    return hipGetLastError();
}

template <int RS, int NF, bool DUMP, bool COUNT>
static hipError_t launch_band_one(hipStream_t st, const BandArgs &a, int grid)
{
    const size_t lds = (size_t)a.b.lds_ints * 4;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)recurrence_band_kernel<RS, NF, DUMP, COUNT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((recurrence_band_kernel<RS, NF, DUMP, COUNT>), dim3(grid), dim3(WAVE * BAND_WAVES), lds, st, a);
    return hipGetLastError();
}

template <int RS>
static hipError_t launch_band_mode(hipStream_t st, const BandArgs &a, int mode, int grid)
{
    const int cells = (a.p.K * RS + WAVE * BAND_WAVES - 1) / (WAVE * BAND_WAVES);    // of a layer, per thread
    switch (mode) {
    case FAST_MODE_PLAN: return launch_band_one<RS, 0, true, false>(st, a, grid);
    case FAST_MODE_COUNT: return launch_band_one<RS, 0, false, true>(st, a, grid);
    default:
        if (cells <= 4) return launch_band_one<RS, 4, false, false>(st, a, grid);
        if (cells <= 8) return launch_band_one<RS, 8, false, false>(st, a, grid);
        return launch_band_one<RS, 0, false, false>(st, a, grid);
    }
}

hipError_t launch_recurrence_band(hipStream_t st, const FastArgs &f, const BandShape &b, const int32_t *recs,
                                  const int32_t *ends, const int32_t *thr, int32_t max_finite, int mode, int grid)
{
    BandArgs a{f.p, b, f.n_lo, f.n_hi, recs, ends, f.sizes, f.cand, f.list, f.n_list_p, f.ticket, f.wave_relax,
               f.chunk_min, f.prune, f.descending, f.Fmin, f.Sbest, f.dummy_idx, f.F_all, f.s_top_p, f.s_bound, thr, max_finite,
               f.whole, f.n_whole_p, f.rest, f.thin, f.leave_out ? 1 : 0, f.B_vals, f.n_B};
    switch (band_row_ints(f.p.D)) {
    case 64: return launch_band_mode<64>(st, a, mode, grid);
    case 128: return launch_band_mode<128>(st, a, mode, grid);
    case 256: return launch_band_mode<256>(st, a, mode, grid);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace alpa
