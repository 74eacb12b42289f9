// Recurrence kernel (Eq. 3): one workgroup of up to sixteen waves per t_max candidate.
//
// Mapping.  Lanes are device counts, and the first layers k are cut into half-blocks of 8.  A batch
// is 16 table entries: the half-block's first layers against a pair of neighbouring columns (last layers
// 2j and 2j + 1) for one submesh shape; it updates the half-block's eight accumulators by
//     acc[k] = min(acc[k], t[k][2j] + F(s-1, 2j+1, d - a), t[k][2j+1] + F(s-1, 2j+2, d - a)),
// 16 additions and 8 three-operand minima for 16 cell-updates per lane.
//
// t_intra is the same for all lanes, but it does not come through the scalar cache: every row of 16 lanes
// loads the batch's 16 entries into ONE vector register (lane l of a row holds entry l), and the addition
// takes its operand from there by a row broadcast (DPP row_newbcast), at the full issue rate of
// the vector unit.  What that gives:
//   * loads return in order and cost one register each, so they run PREFETCH batches ahead; scalar
//     loads return in any order (a wait covers all of them) and cost twenty of the hundred scalar registers
//     a batch, which allows one batch ahead: a lone workgroup of sixteen waves then took 870 clocks
//     per batch and wave, most of it waiting;
//   * the filter t_intra <= t_max is one compare and one select per 16 entries (it was a scalar compare
//     and a scalar select for each), and its mask says whether the batch has anything at all;
//   * rows of 16 lanes need not hold the same entries.  A shape of a devices has cells only for
//     d >= a + s - 1; where those fit in 32 (16) device counts, two (four) neighbouring pairs of columns go
//     through one batch, each in its own half (quarter) of the wave, and meet in the merge.
//     On average half of the lanes would idle otherwise, small meshes almost all of them.
//
// The waves share the work of a layer: wave (wk, wi) owns half-blocks wk and NHB - 1 - wk (together
// the same number of columns for every wk) for its share of the shapes.  Partial minima meet in LDS
// (ds_min).  F(s-1) and F(s) are two buffers of rows F(., first layer, 0..D) with 64 cells of +infinity in
// front of each row, so that the operand of a lane with d - a < 0 needs no mask, and rows of +infinity
// behind the last.  Layer 1 is an ordinary layer whose only finite operand is F(0, K+1, 0) = 0.
//
// Table layout (repack_row_kernel): for every (s - 1, shape q, half-block hb) the pairs of columns from the
// diagonal on, 16 int32 each: [0..7] t_intra of first layers 8hb..8hb+7 for the pair's first column,
// [8..15] for its second; DEV_INF where there is no entry.  `ends` (repack_ends_kernel): for every
// (s - 1, hb, q) the smallest entry of the pairs from each of eight positions on, i.e. behind which
// position a candidate finds nothing any more.
#include "internal.hpp"

namespace alpa {

constexpr int ROW_PAIR = 16;                 // int32 per pair of columns
constexpr int ROW_PAD = 64;                  // +infinity cells in front of d = 0 in an F row
constexpr int ROW_EXTRA = 8;                 // F rows behind first layer K - 1 (a batch reaches 8 columns on)
constexpr int ROW_ENDS = 8;
constexpr int PREFETCH = 4;

// pairs of columns of one (s, q), and how many of them lie in front of half-block hb's
__host__ __device__ constexpr int row_half_blocks(int K) { return (K + 7) / 8; }
__host__ __device__ constexpr int row_pairs_before(int K, int hb)
{
    return hb * ((K + 1) / 2) - 2 * hb * (hb - 1);
}
__host__ __device__ constexpr int row_pairs(int K) { return row_pairs_before(K, row_half_blocks(K)); }
// position (in pairs behind the diagonal) from which `ends` entry j counts
__host__ __device__ constexpr int row_end_pos(int K, int j)
{
    const int scale = K <= 64 ? 1 : K <= 128 ? 2 : 4;
    return scale * (j <= 4 ? 2 * j : j == 5 ? 12 : j == 6 ? 16 : 24);
}

size_t row_table_ints(int K, int Smax, int S)
{
    return ((size_t)Smax * S * row_pairs(K) + 64) * ROW_PAIR;
}
size_t row_ends_ints(int K, int Smax, int S) { return (size_t)Smax * row_half_blocks(K) * S * ROW_ENDS; }

// one thread per (s, q, hb, pair) and half of the pair
__global__ void repack_row_kernel(const int32_t *__restrict__ table, int K, int S, long long n,
                                  int32_t *__restrict__ recs)
{
    const int P = row_pairs(K), NHB = row_half_blocks(K);
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
         e += (long long)gridDim.x * blockDim.x) {
        const int u = (int)(e & (ROW_PAIR - 1));
        const long long r = e >> 4;
        const int pair = (int)(r % P);
        const long long sq = r / P;
        const int q = (int)(sq % S);
        const long long s = sq / S;
        int hb = 0;
        while (hb + 1 < NHB && row_pairs_before(K, hb + 1) <= pair) ++hb;
        const int i = 8 * hb + 2 * (pair - row_pairs_before(K, hb)) + (u >> 3);
        const int k = 8 * hb + (u & 7);
        int32_t v = DEV_INF;
        if (i < K && k <= i) {
            const int32_t t = table[((s * K + k) * K + i) * S + q];
            if (t != INF_I32) v = t;
        }
        recs[e] = v;
    }
}

__global__ void repack_row_pad_kernel(int32_t *__restrict__ p, int n)
{
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x)
        p[x] = DEV_INF;
}

// a wave per (s, hb, q): lanes over the pairs, a minimum per position
__global__ __launch_bounds__(256) void repack_ends_kernel(const int32_t *__restrict__ recs, int K, int S,
                                                          int n, int32_t *__restrict__ ends)
{
    const int NHB = row_half_blocks(K), P = row_pairs(K);
    const int lane = threadIdx.x & (WAVE - 1);
    const int n_waves = gridDim.x * (blockDim.x / WAVE);
    for (int e = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6); e < n; e += n_waves) {
        const int q = e % S, hb = (e / S) % NHB, s = e / (S * NHB);
        const int pairs = (K + 1) / 2 - 4 * hb;
        const int32_t *row = recs + (((size_t)s * S + q) * P + row_pairs_before(K, hb)) * ROW_PAIR;
        int32_t mn[ROW_ENDS];
#pragma unroll
        for (int j = 0; j < ROW_ENDS; ++j) mn[j] = DEV_INF;
        for (int x = lane; x < pairs * ROW_PAIR; x += WAVE) {
            const int32_t v = row[x];
            const int pos = x / ROW_PAIR;
#pragma unroll
            for (int j = 0; j < ROW_ENDS; ++j)
                if (pos >= row_end_pos(K, j)) mn[j] = min(mn[j], v);
        }
#pragma unroll
        for (int j = 0; j < ROW_ENDS; ++j) {
            const int32_t m = wave_min_i32(mn[j]);
            if (lane == j) ends[(size_t)e * ROW_ENDS + j] = m;
        }
    }
}

hipError_t launch_repack_row(hipStream_t st, const int32_t *table, int K, int Smax, int S,
                             int32_t *recs, int32_t *ends)
{
    const long long n = (long long)Smax * S * row_pairs(K) * ROW_PAIR;
    hipLaunchKernelGGL(repack_row_pad_kernel, dim3(4), dim3(256), 0, st, recs + n, 64 * ROW_PAIR);
    hipLaunchKernelGGL(repack_row_kernel, dim3((unsigned)std::min<long long>((n + 255) / 256, 16384)),
                       dim3(256), 0, st, table, K, S, n, recs);
    const int ne = Smax * row_half_blocks(K) * S;
    hipLaunchKernelGGL(repack_ends_kernel, dim3(std::min((ne + 3) / 4, 8192)), dim3(256), 0, st, recs, K, S,
                       ne, ends);
    return hipGetLastError();
}

// entry N of the row's 16
template <int N>
__device__ __forceinline__ int32_t row_entry(int32_t t)
{
    return __builtin_amdgcn_update_dpp(0, t, 0x150 + N, 0xf, 0xf, true);
}

template <int U>
__device__ __forceinline__ void row_update(int32_t (&acc)[8], int32_t t, int32_t fX, int32_t fY)
{
    // four rows at a time: eight sums in flight before their minima
    const int32_t x0 = row_entry<U>(t) + fX, y0 = row_entry<U + 8>(t) + fY;
    const int32_t x1 = row_entry<U + 1>(t) + fX, y1 = row_entry<U + 9>(t) + fY;
    const int32_t x2 = row_entry<U + 2>(t) + fX, y2 = row_entry<U + 10>(t) + fY;
    const int32_t x3 = row_entry<U + 3>(t) + fX, y3 = row_entry<U + 11>(t) + fY;
    acc[U] = min(acc[U], min(x0, y0));
    acc[U + 1] = min(acc[U + 1], min(x1, y1));
    acc[U + 2] = min(acc[U + 2], min(x2, y2));
    acc[U + 3] = min(acc[U + 3], min(x3, y3));
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int wave_prefix_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // last lane of rows 0, 2 to rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // lane 31 to rows 2, 3
    return v;
}

__device__ __forceinline__ bool row_can_skip(const int64_t *chunk_min, int j, int32_t c, int B, int lane)
{
    const int g = j / PRUNE_CHUNK;
    int64_t m = INF_I64;
    for (int x = lane; x < g; x += WAVE)
        m = min64(m, __atomic_load_n(&chunk_min[x], __ATOMIC_RELAXED));
    m = wave_min_i64(m);
    return m != INF_I64 && (int64_t)B * (int64_t)c >= m;
}

struct RowArgs {
    Problem p;
    int NHB, NWK, WI;        // half-blocks; waves along them (ceil(NHB / 2)); wave groups over the shapes
    const int32_t *recs, *ends, *sizes, *cand, *list, *n_list_p;
    int32_t *ticket;
    unsigned long long *wave_relax;
    int64_t *chunk_min;
    int prune, descending;
    int32_t *Fmin, *Sbest;
    int dummy_idx;
    int32_t *F_all;
    const int32_t *s_top_p, *s_bound;
};

// RS: int32 per F row (ROW_PAD + 1 + device counts of the size class).  DUMP: store every layer to F_all
// (plan recovery: entry j of the list is candidate j itself, and only what the walk back from layer
// s_top_p[j] can reach is computed).  COUNT: tally the executed updates.
template <int RS, bool DUMP, bool COUNT>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(7)))
void recurrence_row_kernel(RowArgs a)
{
    extern __shared__ int32_t lds[];                   // F [2][K + ROW_EXTRA][RS], then the lengths
    __shared__ int32_t sh_tk[1];
    __shared__ int32_t sh_skip[16];
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = a.p.K, D = a.p.D, S = a.p.S, NHB = a.NHB, NWK = a.NWK, WI = a.WI;
    const int nw = NWK * WI;
    const int wk = wid % NWK, wi = wid / NWK;
    const int LS = (K + 2) * (D + 1);
    const int BUF = (K + ROW_EXTRA) * RS;
    const int P = row_pairs(K);
    uint8_t *lens = (uint8_t *)(lds + 2 * BUF);        // [s - 1][hb][q]: pairs with an entry for the candidate
    const int size_of_lane = a.sizes[min(lane, S - 1)];                   // lane q holds a_q (S <= 64)
    const int n = __builtin_amdgcn_readfirstlane(*a.n_list_p);
    const int hf_end = 2 * ((D + WAVE - 1) / WAVE);
    const unsigned inv_WI = ((1u << 20) + WI - 1) / WI;                   // x / WI = x * inv_WI >> 20 for x < 2^20 / WI
    unsigned long long rows_total = 0;

    for (;;) {
        const int tk = draw_ticket(a.ticket, tid, sh_tk);
        if (tk >= n) break;                            // the workgroup's only exit
        const int pos = a.descending ? n - 1 - tk : tk;
        const int j = DUMP ? pos : __builtin_amdgcn_readfirstlane(a.list[pos]);
        const int32_t c_given = __builtin_amdgcn_readfirstlane(a.cand[j]);
        const int32_t c = min(c_given, DEV_INF - 1);   // the sentinel entries pass no candidate
        if (a.prune) {
            sh_skip[wid] = row_can_skip(a.chunk_min, j, c_given, a.p.B, lane) ? 1 : 0;
            __syncthreads();
            const int skip = __builtin_amdgcn_readfirstlane(sh_skip[0]);
            __syncthreads();
            if (skip) {
                a.Fmin[j] = DEV_INF;                   // all threads, same value
                a.Sbest[j] = -1;
                continue;
            }
        }
        // Plan recovery walks back from F(s*, first layer 1, all devices): only layers up to s* are needed,
        // and of layer s only first layers (0-based) >= s* - s
        const int s_top = DUMP ? min(a.p.Smax, __builtin_amdgcn_readfirstlane(a.s_top_p[j])) : a.p.Smax;
        int32_t *F_out = DUMP ? a.F_all + (size_t)j * (size_t)(a.p.Smax + 1) * LS : nullptr;
        if (DUMP)                                      // layer 0: only F(0, K+1, 0) = 0
            for (int x = tid; x < LS; x += blockDim.x) F_out[x] = (x == (K + 1) * (D + 1)) ? 0 : DEV_INF;
        for (int x = tid; x < 2 * BUF; x += blockDim.x) lds[x] = (x == K * RS + ROW_PAD) ? 0 : DEV_INF;
        // how many pairs behind the diagonal have an entry for the candidate, to the grain of `ends`
        for (int x = tid; x < s_top * NHB * S; x += blockDim.x) {
            const int4 *e = (const int4 *)(a.ends + (size_t)x * ROW_ENDS);
            const int4 e0 = e[0], e1 = e[1];
            int len = 0;
            len += e0.x <= c ? row_end_pos(K, 1) - row_end_pos(K, 0) : 0;
            len += e0.y <= c ? row_end_pos(K, 2) - row_end_pos(K, 1) : 0;
            len += e0.z <= c ? row_end_pos(K, 3) - row_end_pos(K, 2) : 0;
            len += e0.w <= c ? row_end_pos(K, 4) - row_end_pos(K, 3) : 0;
            len += e1.x <= c ? row_end_pos(K, 5) - row_end_pos(K, 4) : 0;
            len += e1.y <= c ? row_end_pos(K, 6) - row_end_pos(K, 5) : 0;
            len += e1.z <= c ? row_end_pos(K, 7) - row_end_pos(K, 6) : 0;
            len += e1.w <= c ? 128 - row_end_pos(K, 7) : 0;
            lens[x] = (uint8_t)len;
        }
        __syncthreads();
        int32_t best = DEV_INF, sbest = 0;
        unsigned rows = 0;

        // A stream: batches of one form (one, two or four pairs of columns) for one of the wave's half-blocks
        // and one window of 64 device counts (the top one ends at D).  The batches of a (half-block,
        // window), shape after shape, are dealt to the wave groups in equal shares.  prepare() goes to the
        // wave's next stream, which may be in a later layer, and sends its first entries on their way: they need
        // nothing of the layer before, so that happens ahead of the barrier.
        int st_s = 1, st_hf = -1;                      // layer; 2 * window + half
        unsigned long long shapes = 0, todo = 0;       // shapes left in (st_s, st_hf); in the stream
        int mode_l = 0, begin_l = 0, count_l = 0;      // lane q: form, first batch and batches of the wave's share
        int left_all = 0, mode = 0, out_row = 0;
        const char *recs_w = nullptr;                  // records of the half-block, layer st_s, shape 0
        int t_off = 0, f_off = 0, left = 0, t_step = 0, f_step = 0, f_base = 0;
        int t_lane = 0, f_lane = 0;                    // lane parts of the addresses (bytes / cells)
        int32_t t[PREFETCH], fX[PREFETCH], fY[PREFETCH];
        auto open = [&]() {                            // next shape of the stream
            const int q = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int b = __builtin_amdgcn_readlane(begin_l, q);
            left = __builtin_amdgcn_readlane(count_l, q);
            t_off = q * P * (ROW_PAIR * 4) + b * t_step;
            f_off = f_base - __builtin_amdgcn_readlane(size_of_lane, q) + b * f_step;
        };
        auto advance = [&]() {
            if (--left > 0) {
                t_off += t_step;
                f_off += f_step;
            } else if (todo) {
                open();
            } else {                                   // nothing further: stay
                left = 1 << 30;
                t_step = f_step = 0;
            }
        };
        int hb = 0, top = 0, first = 0;
        auto prepare = [&]() {
            while (shapes == 0) {
                if (++st_hf >= hf_end) {
                    st_hf = 0;
                    if (++st_s > s_top) return;
                }
                const int h = st_hf & 1;
                hb = h ? NHB - 1 - wk : wk;
                if ((h && hb == wk) || (DUMP && 8 * hb + 7 < s_top - st_s)) continue;
                top = D - WAVE * (st_hf >> 1);
                const int rem = top - size_of_lane - st_s + 2;  // device counts the shape serves in the window
                mode_l = rem > 32 ? 0 : rem > 16 ? 1 : 2;
                const int len = lens[((st_s - 1) * NHB + hb) * S + min(lane, S - 1)];
                // the last layer of a stage is at most K - s; in layer 1 it is K - 1 and nothing else
                first = st_s == 1 ? (K - 1) / 2 - 4 * hb : 0;
                const int pairs = st_s == 1 ? (len > first ? 1 : 0) : min(len, max(0, K - st_s + 2 - 8 * hb) >> 1);
                const bool alive = lane < S && rem > 0;
                const int batches = alive ? (pairs + (1 << mode_l) - 1) >> mode_l : 0;
                const int upto = wave_prefix_sum(batches);
                const int total = __builtin_amdgcn_readlane(upto, WAVE - 1);
                // this wave's share of the total; batches of lane q's shape in it
                const int lo = (int)(((unsigned long long)(unsigned)(total * wi) * inv_WI) >> 20);
                const int hi = (int)(((unsigned long long)(unsigned)(total * (wi + 1)) * inv_WI) >> 20);
                begin_l = max(0, lo - (upto - batches));
                count_l = min(batches, hi - (upto - batches)) - begin_l;
                shapes = __ballot(count_l > 0);
            }
            mode = __builtin_amdgcn_readlane(mode_l, __builtin_ctzll(shapes));
            todo = shapes & __ballot(mode_l == mode);
            shapes &= ~todo;
            left_all = 0;
            for (unsigned long long x = todo; x; x &= x - 1)
                left_all += __builtin_amdgcn_readlane(count_l, __builtin_ctzll(x));
            recs_w = (const char *)(a.recs + ((size_t)(st_s - 1) * S * P + row_pairs_before(K, hb) + first) * ROW_PAIR);
            t_step = (ROW_PAIR * 4) << mode;
            f_step = (2 * RS) << mode;
            const int width = WAVE >> mode;
            const int sub = lane >> (6 - mode);
            const int cell = ROW_PAD + top + 1 - width + (lane & (width - 1));  // the lane's cell in an F row
            out_row = 8 * hb * RS + cell;
            t_lane = (lane & 15) * 4 + sub * (ROW_PAIR * 4);
            f_lane = (sub * 2) * RS + cell;
            f_base = (8 * hb + 2 * first + 1) * RS;
            open();
#pragma unroll
            for (int x = 0; x < PREFETCH; ++x) {
                t[x] = *(const int32_t *)(recs_w + (uint32_t)t_off + (uint32_t)t_lane);
                fX[x] = f_lane + f_off;                // where the operands are; read behind the barrier
                advance();
            }
        };
        prepare();
        for (int s = 1; s <= s_top; ++s) {
            const int32_t *Fp = lds + ((s - 1) & 1) * BUF;
            int32_t *Fn = lds + (s & 1) * BUF;
            // (the other buffer's last readers have passed the barrier at the end of the last layer)
            for (int r = wid; r < K; r += nw)
                for (int x = lane; x < D; x += WAVE) Fn[r * RS + ROW_PAD + 1 + x] = DEV_INF;
            Fn[K * RS + ROW_PAD] = DEV_INF;            // F(s, K+1, 0) for s >= 1
            __syncthreads();
            while (st_s == s) {
                int32_t acc[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[u] = DEV_INF;
#pragma unroll
                for (int x = 0; x < PREFETCH; ++x) {
                    const int32_t *f = Fp + fX[x];
                    fX[x] = f[0];
                    fY[x] = f[RS];
                }
#pragma nounroll
                for (; left_all > 0; left_all -= PREFETCH) {
#pragma unroll
                    for (int x = 0; x < PREFETCH; ++x) {
                        const int32_t lim = left_all > x ? c : -1;
                        const bool pass = t[x] <= lim;
                        if (__ballot(pass)) {
                            const int32_t tv = pass ? t[x] : DEV_INF;
                            row_update<0>(acc, tv, fX[x], fY[x]);
                            row_update<4>(acc, tv, fX[x], fY[x]);
                            if (COUNT) rows += 16;
                        }
                        t[x] = *(const int32_t *)(recs_w + (uint32_t)t_off + (uint32_t)t_lane);
                        const int32_t *f = Fp + (f_lane + f_off);
                        fX[x] = f[0];
                        fY[x] = f[RS];
                        advance();
                    }
                }
                int32_t *out = Fn + out_row;
                prepare();
#pragma unroll
                for (int u = 0; u < 8; ++u) atomicMin(&out[u * RS], acc[u]);
            }
            __syncthreads();
            const int32_t f1 = Fn[ROW_PAD + D];        // F(s, first layer, all devices)
            if (f1 < best) { best = f1; sbest = s; }   // lowest s on ties
            if (!DUMP && a.s_bound[s] >= __builtin_amdgcn_readfirstlane(best)) break;
            if (DUMP) {
                int32_t *Fs = F_out + (size_t)s * LS;
                for (int r = wid; r <= K; r += nw)
                    for (int x = lane; x <= D; x += WAVE) Fs[(r + 1) * (D + 1) + x] = Fn[r * RS + ROW_PAD + x];
            }
        }
        const int32_t bv = __builtin_amdgcn_readfirstlane(best);
        const int slot = wid == 0 ? j : a.dummy_idx;   // wave 0 owns the result
        a.Fmin[slot] = bv;                             // all lanes, same value
        a.Sbest[slot] = bv >= DEV_INF ? 0 : __builtin_amdgcn_readfirstlane(sbest);
        if (a.prune && bv < DEV_INF)                   // uniform
            publish_min(&a.chunk_min[j / PRUNE_CHUNK], (int64_t)bv + (int64_t)(a.p.B - 1) * (int64_t)c_given, tid);
        if (COUNT) rows_total += rows;
        __syncthreads();                               // LDS is reused by the next candidate
    }
    if (COUNT) atomicAdd(a.wave_relax, lane == 0 ? rows_total : 0ull);
}

// F rows of the size class that holds D devices (0: none does)
static constexpr int row_ints(int D)
{
    return D <= 16 ? 81 : D <= 32 ? 97 : D <= 64 ? 129 : D <= 128 ? 193 : D <= 256 ? 321 : 0;
}
static size_t row_lds(int K, int D, int S)
{
    return (size_t)2 * (K + ROW_EXTRA) * row_ints(D) * sizeof(int32_t) +
           (size_t)std::min(K, D) * row_half_blocks(K) * S;
}

// Sizes whose two F buffers fit a compute unit's LDS (160 KiB, less the kernel's few static words)
bool row_serves(int K, int D, int S) { return row_ints(D) != 0 && row_lds(K, D, S) <= 160 * 1024 - 256; }

// waves along the half-blocks and wave groups over the shapes: up to sixteen waves
static void row_waves(int K, int S, int &NWK, int &WI)
{
    NWK = (row_half_blocks(K) + 1) / 2;
    WI = std::max(1, std::min(16 / NWK, S));
}

int row_blocks_per_cu(int K, int D, int S)
{
    int NWK, WI;
    row_waves(K, S, NWK, WI);
    return std::max(1, std::min((int)((160 * 1024) / (row_lds(K, D, S) + 256)), 32 / (NWK * WI)));
}

template <int RS, bool DUMP, bool COUNT>
static hipError_t launch_row_one(hipStream_t st, const RowArgs &a, int grid, size_t lds)
{
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)recurrence_row_kernel<RS, DUMP, COUNT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((recurrence_row_kernel<RS, DUMP, COUNT>), dim3(grid), dim3(WAVE * a.NWK * a.WI), lds,
                       st, a);
    return hipGetLastError();
}

template <int RS>
static hipError_t launch_row_mode(hipStream_t st, const RowArgs &a, int mode, int grid, size_t lds)
{
    switch (mode) {
    case FAST_MODE_PLAN: return launch_row_one<RS, true, false>(st, a, grid, lds);
    case FAST_MODE_COUNT: return launch_row_one<RS, false, true>(st, a, grid, lds);
    default: return launch_row_one<RS, false, false>(st, a, grid, lds);
    }
}

hipError_t launch_recurrence_row(hipStream_t st, const FastArgs &f, const int32_t *recs,
                                 const int32_t *ends, int mode, int grid)
{
    int NWK, WI;
    row_waves(f.p.K, f.p.S, NWK, WI);
    RowArgs a{f.p, row_half_blocks(f.p.K), NWK, WI, recs, ends, f.sizes, f.cand, f.list, f.n_list_p, f.ticket, f.wave_relax,
              f.chunk_min, f.prune, f.descending, f.Fmin, f.Sbest, f.dummy_idx, f.F_all, f.s_top_p, f.s_bound};
    const size_t lds = row_lds(f.p.K, f.p.D, f.p.S);
    switch (row_ints(f.p.D)) {
    case 81: return launch_row_mode<81>(st, a, mode, grid, lds);
    case 97: return launch_row_mode<97>(st, a, mode, grid, lds);
    case 129: return launch_row_mode<129>(st, a, mode, grid, lds);
    case 193: return launch_row_mode<193>(st, a, mode, grid, lds);
    case 321: return launch_row_mode<321>(st, a, mode, grid, lds);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace alpa
