// Candidate preparation on the device: the "SortedAndFilter(t_intra, epsilon)" step of
// Alg. 1.  Latencies are integer microseconds and epsilon is 1 us (Sec. 5.2, performance
// optimisation #1), so the step is: ascending order, duplicates removed.
//
// Kernels: gather of the table's values, a least-significant-digit radix sort (8-bit
// digits, one wave per slice, stable ranking inside a wave by ballot matching), adjacent
// -difference flags + scan + compaction, quantile pick, and rank lookup for the caller's
// own candidate order.
#include "internal.hpp"

namespace alpa {

constexpr int SORT_BLOCKS = SORT_SLICES;   // one wave each, contiguous slice per wave
constexpr int RADIX = SORT_RADIX;

// ---------------------------------------------------------------- gather

// One key per table entry with last layer >= first layer, at a fixed position, so that
// the number of keys is known on the host; +infinity becomes `inf_key` (largest finite
// value + 1) and is dropped again after the sort.
__global__ void gather_table_values_kernel(const int32_t *__restrict__ table, int K, int S,
                                           int32_t inf_key, int32_t *__restrict__ keys)
{
    const long long total = (long long)K * K * K * S;
    const int P = K * (K + 1) / 2;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        int q = (int)(e % S);
        long long r = e / S;
        int i = (int)(r % K); r /= K;
        int k = (int)(r % K);
        int s = (int)(r / K);
        if (i < k) continue;
        int tri = k * K - (k * (k - 1)) / 2 + (i - k);
        int32_t t = table[e];
        keys[((long long)s * P + tri) * S + q] = (t == INF_I32) ? inf_key : t;
    }
}

// ---------------------------------------------------------------- radix sort

__device__ __forceinline__ void slice_of(int n, int b, int &lo, int &hi)
{
    int per = (n + SORT_BLOCKS - 1) / SORT_BLOCKS;
    per = (per + WAVE - 1) / WAVE * WAVE;
    lo = min(n, b * per);
    hi = min(n, lo + per);
}

__global__ __launch_bounds__(WAVE) void radix_hist_kernel(const int32_t *__restrict__ keys, int n,
                                                          int shift, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t cnt[RADIX];
    const int lane = threadIdx.x;
    for (int x = lane; x < RADIX; x += WAVE) cnt[x] = 0;
    __syncthreads();
    int lo, hi;
    slice_of(n, blockIdx.x, lo, hi);
    for (int j = lo + lane; j < hi; j += WAVE) {
        uint32_t dgt = ((uint32_t)keys[j] >> shift) & (RADIX - 1);
        atomicAdd(&cnt[dgt], 1u);
    }
    __syncthreads();
    for (int x = lane; x < RADIX; x += WAVE) hist[x * SORT_BLOCKS + blockIdx.x] = cnt[x];
}

// Exclusive scan of `len` uint32 values in place, one block of 1024 threads: every thread
// owns a contiguous segment.
__global__ __launch_bounds__(1024) void scan_u32_kernel(uint32_t *__restrict__ v, int len,
                                                        uint32_t *__restrict__ total_out)
{
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int L = (len + 1023) / 1024;
    const int lo = min(len, t * L), hi = min(len, lo + L);
    uint32_t s = 0;
    for (int j = lo; j < hi; ++j) s += v[j];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint32_t o = (t >= off) ? part[t - off] : 0u;
        __syncthreads();
        part[t] += o;
        __syncthreads();
    }
    uint32_t run = part[t] - s;
    for (int j = lo; j < hi; ++j) {
        uint32_t x = v[j];
        v[j] = run;
        run += x;
    }
    if (total_out && t == 1023) *total_out = part[1023];
}

// Offsets of one radix pass from the per-slice digit counts hist[digit][slice]: one block per
// digit scans its SORT_BLOCKS counts in place (exclusive) and leaves the digit's total in
// totals[digit]; digit_base_kernel then scans the 256 totals.
__global__ __launch_bounds__(SORT_BLOCKS) void digit_scan_kernel(uint32_t *__restrict__ hist,
                                                                 uint32_t *__restrict__ totals)
{
    __shared__ uint32_t part[SORT_BLOCKS];
    const int t = threadIdx.x;
    uint32_t *row = hist + blockIdx.x * SORT_BLOCKS;
    const uint32_t own = row[t];
    part[t] = own;
    __syncthreads();
    for (int off = 1; off < SORT_BLOCKS; off <<= 1) {
        const uint32_t o = (t >= off) ? part[t - off] : 0u;
        __syncthreads();
        part[t] += o;
        __syncthreads();
    }
    row[t] = part[t] - own;
    if (t == SORT_BLOCKS - 1) totals[blockIdx.x] = part[t];
}

__global__ __launch_bounds__(RADIX) void digit_base_kernel(uint32_t *__restrict__ totals)
{
    __shared__ uint32_t part[RADIX];
    const int t = threadIdx.x;
    const uint32_t own = totals[t];
    part[t] = own;
    __syncthreads();
    for (int off = 1; off < RADIX; off <<= 1) {
        const uint32_t o = (t >= off) ? part[t - off] : 0u;
        __syncthreads();
        part[t] += o;
        __syncthreads();
    }
    totals[t] = part[t] - own;
}

__global__ __launch_bounds__(WAVE) void radix_scatter_kernel(const int32_t *__restrict__ keys_in,
                                                             int32_t *__restrict__ keys_out, int n,
                                                             int shift,
                                                             const uint32_t *__restrict__ offs,
                                                             const uint32_t *__restrict__ digit_base)
{
    __shared__ uint32_t base[RADIX];
    const int lane = threadIdx.x;
    for (int x = lane; x < RADIX; x += WAVE)
        base[x] = digit_base[x] + offs[x * SORT_BLOCKS + blockIdx.x];
    __syncthreads();
    int lo, hi;
    slice_of(n, blockIdx.x, lo, hi);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int j0 = lo; j0 < hi; j0 += WAVE) {
        const int j = j0 + lane;
        const bool valid = j < hi;
        const int32_t key = valid ? keys_in[j] : 0;
        const uint32_t dgt = ((uint32_t)key >> shift) & (RADIX - 1);
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (dgt >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            m &= bit ? bal : ~bal;
        }
        const uint32_t rank = (uint32_t)__popcll(m & lt);
        uint32_t pos = 0;
        if (valid) pos = base[dgt] + rank;
        __syncthreads();
        if (valid && rank == 0) base[dgt] += (uint32_t)__popcll(m);
        __syncthreads();
        if (valid) keys_out[pos] = key;
    }
}

// ---------------------------------------------------------------- dedup

constexpr int DEDUP_TILE = 1024 * 4;

__device__ __forceinline__ uint32_t head_flag(const int32_t *keys, int j, int n, int32_t drop_key)
{
    if (j >= n) return 0u;
    const int32_t x = keys[j];
    if (x == drop_key) return 0u;
    return (j == 0 || keys[j - 1] != x) ? 1u : 0u;
}

__global__ __launch_bounds__(1024) void dedup_count_kernel(const int32_t *__restrict__ keys, int n,
                                                           int32_t drop_key,
                                                           uint32_t *__restrict__ block_cnt)
{
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x;
    const int base = blockIdx.x * DEDUP_TILE + t * 4;
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) c += head_flag(keys, base + u, n, drop_key);
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((t & 63) == 0) wsum[t >> 6] = c;
    __syncthreads();
    if (t == 0) {
        uint32_t s = 0;
        for (int w = 0; w < 16; ++w) s += wsum[w];
        block_cnt[blockIdx.x] = s;
    }
}

__global__ __launch_bounds__(1024) void dedup_write_kernel(const int32_t *__restrict__ keys, int n,
                                                           int32_t drop_key,
                                                           const uint32_t *__restrict__ block_off,
                                                           int32_t *__restrict__ unique)
{
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int base = blockIdx.x * DEDUP_TILE + t * 4;
    uint32_t f[4], c = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) { f[u] = head_flag(keys, base + u, n, drop_key); c += f[u]; }
    part[t] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint32_t o = (t >= off) ? part[t - off] : 0u;
        __syncthreads();
        part[t] += o;
        __syncthreads();
    }
    uint32_t pos = block_off[blockIdx.x] + part[t] - c;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (f[u]) unique[pos++] = keys[base + u];
}

// ---------------------------------------------------------------- distinct values by bitmap
//
// SortedAndFilter of Alg. 1 for tables whose finite values are small integers: instead of sorting every entry, each finite
// entry sets one bit of a presence bitmap and the set bits are listed in order; the result is the same ascending list
// of distinct values.

__global__ void bitmap_clear_kernel(uint32_t *__restrict__ bm, int words)
{
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < words; x += gridDim.x * blockDim.x)
        bm[x] = 0u;
}

// A thread takes a stage and shape for eight numbers of stages behind it, with all loads in flight, and leaves out what
// repeats the one before: of a model whose stages run at their fastest wherever they fit, most entries do.  LOCAL: a block
// marks a bitmap of its own in LDS and then merges the words it touched into the global one (up to 64 KiB); else the
// global one is marked directly.  Bound by reading the table (128 layers on 8 x 8, 126 MB: 80 us with
// an entry at a time).
template <bool LOCAL>
__global__ __launch_bounds__(1024) void bitmap_mark_kernel(const int32_t *__restrict__ table, int K,
                                                           int S, int words,
                                                           uint32_t *__restrict__ bm)
{
    extern __shared__ uint32_t lbm[];             // [words] if LOCAL
    if (LOCAL) {
        for (int x = threadIdx.x; x < words; x += blockDim.x) lbm[x] = 0u;
        __syncthreads();
    }
    const int n = K * K * S, total = n * ((K + 7) / 8);    // (256 layers, 64 shapes: 1.3e8)
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < total; x += gridDim.x * blockDim.x) {
        const int ch = x / n, e = x - ch * n, r = e / S, k = r / K;
        if (r - k * K < k) continue;               // (last layer in front of the first)
        const int32_t *t = table + (size_t)ch * 8 * n + e;
        int32_t v[8], prev = INF_I32;
#pragma unroll
        for (int y = 0; y < 8; ++y) v[y] = ch * 8 + y < K ? t[(size_t)y * n] : INF_I32;
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            if (v[y] != INF_I32 && v[y] != prev) {
                const uint32_t bit = 1u << (v[y] & 31);
                if (!LOCAL) atomicOr(&bm[v[y] >> 5], bit);
                else if (!(lbm[v[y] >> 5] & bit)) atomicOr(&lbm[v[y] >> 5], bit);   // a stale 0 only costs the atomic
            }
            prev = v[y];
        }
    }
    if (!LOCAL) return;
    __syncthreads();
    for (int x = threadIdx.x; x < words; x += blockDim.x) {
        const uint32_t v = lbm[x];
        if (v && (v & ~__atomic_load_n(&bm[x], __ATOMIC_RELAXED))) atomicOr(&bm[x], v);
    }
}

__global__ __launch_bounds__(1024) void bitmap_count_kernel(const uint32_t *__restrict__ bm,
                                                            int words,
                                                            uint32_t *__restrict__ block_cnt)
{
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x;
    const int x = blockIdx.x * 1024 + t;
    uint32_t c = x < words ? __popc(bm[x]) : 0u;
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((t & 63) == 0) wsum[t >> 6] = c;
    __syncthreads();
    if (t == 0) {
        uint32_t s = 0;
        for (int w = 0; w < 16; ++w) s += wsum[w];
        block_cnt[blockIdx.x] = s;
    }
}

// Lists the bits of words [1024 b, 1024 b + 1024) behind those of the words in front, which the block counts itself: from the
// blocks' counts, or from the words where they are few (up to 16 blocks: one launch instead of three).
__global__ __launch_bounds__(1024) void bitmap_write_kernel(const uint32_t *__restrict__ bm,
                                                            int words,
                                                            const uint32_t *__restrict__ block_cnt, int counted,
                                                            int32_t *__restrict__ unique,
                                                            uint32_t *__restrict__ n_unique)
{
    __shared__ uint32_t wsum[16], wfront[16];
    const int t = threadIdx.x, lane = t & 63;
    const int x = blockIdx.x * 1024 + t;
    uint32_t w = x < words ? bm[x] : 0u, front = 0;
    if (counted)
        for (int b = t; b < (int)blockIdx.x; b += 1024) front += block_cnt[b];
    else
        for (int y = t; y < (int)blockIdx.x * 1024; y += 1024) front += __popc(bm[y]);
    const uint32_t c = __popc(w);
    uint32_t upto = c;                             // bits up to this lane's word
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(upto, off, 64);
        if (lane >= off) upto += o;
    }
    for (int off = 32; off >= 1; off >>= 1) front += __shfl_xor(front, off, 64);
    if (lane == 63) { wsum[t >> 6] = upto; wfront[t >> 6] = front; }
    __syncthreads();
    uint32_t pos = upto - c;
    for (int y = 0; y < 16; ++y) pos += wfront[y] + (y < (t >> 6) ? wsum[y] : 0u);
    if (blockIdx.x == gridDim.x - 1 && t == 1023) *n_unique = pos + c;
    while (w) {                                   // set bits, lowest first
        const int b = __ffs(w) - 1;
        unique[pos++] = (x << 5) + b;
        w &= w - 1;
    }
}

// ---------------------------------------------------------------- short lists
//
// A caller's list of up to LIST_SORT_MAX values in one block: sorted in LDS (bitonic), the first of each run kept, and every
// value's place among them (rank_of_orig, if wanted).  The value -1 is no candidate and has no place (-1), as in the radix sort
// of longer lists; it sorts behind all others, with what fills up the keys.  1500 values: 16 launches of the radix sort take
// 55 us, and it three more for the places.
__global__ __launch_bounds__(1024) void list_sort_kernel(const int32_t *__restrict__ tmax, int n, int N2,
                                                         int32_t *__restrict__ unique, uint32_t *__restrict__ n_unique,
                                                         SolveState *state, int32_t *__restrict__ rank_of_orig)
{
    extern __shared__ uint32_t keys[];             // [N2] keys, [N2] their places among the distinct ones
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x, lane = t & 63;
    uint32_t *const place = keys + N2;
    for (int x = t; x < N2; x += 1024) keys[x] = x < n ? (uint32_t)tmax[x] : ~0u;
    __syncthreads();
    for (int size = 2; size <= N2; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int x = t; x < N2 / 2; x += 1024) {
                const int lo = 2 * x - (x & (stride - 1)), hi = lo + stride;
                const uint32_t a = keys[lo], b = keys[hi];
                if ((a > b) == ((lo & size) == 0)) { keys[lo] = b; keys[hi] = a; }
            }
            // pairs up to 64 apart stay in the 128 keys of one wave, also in the next step
            const int next = stride > 1 ? stride >> 1 : size;
            if (max(stride, next) > 64) __syncthreads();
            else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
            }
        }
    __syncthreads();
    const int per = (N2 + 1023) / 1024, from = t * per;    // (N2 is a power of two: 1, 2, 4 or 8)
    uint32_t c = 0;
    for (int x = from; x < min(from + per, n); ++x) c += keys[x] != ~0u && (x == 0 || keys[x - 1] != keys[x]);
    uint32_t upto = c;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(upto, off, 64);
        if (lane >= off) upto += o;
    }
    if (lane == 63) wsum[t >> 6] = upto;
    __syncthreads();
    uint32_t pos = upto - c, all = 0;
    for (int y = 0; y < 16; ++y) {
        if (y < (t >> 6)) pos += wsum[y];
        all += wsum[y];
    }
    for (int x = from; x < min(from + per, n); ++x) {
        const bool head = keys[x] != ~0u && (x == 0 || keys[x - 1] != keys[x]);
        if (head) unique[pos++] = (int32_t)keys[x];
        place[x] = keys[x] != ~0u ? pos - 1 : ~0u;
    }
    if (t == 0) {
        *n_unique = all;
        state->n_cand = (int)all;
        state->n_distinct = (int)all;
    }
    if (!rank_of_orig) return;
    __syncthreads();
    for (int j = t; j < n; j += 1024) {
        const uint32_t v = (uint32_t)tmax[j];
        int lo = 0, hi = n - 1;                    // the first key that is not below (there is one)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (keys[mid] < v) lo = mid + 1; else hi = mid;
        }
        rank_of_orig[j] = (int32_t)place[lo];
    }
}

// ---------------------------------------------------------------- candidate lists

// rank_of_orig[j] = index of tmax[j] in the distinct list (binary search; it ascends as unsigned)
__global__ void rank_lookup_kernel(const int32_t *__restrict__ tmax, int n,
                                   const int32_t *__restrict__ unique,
                                   const uint32_t *__restrict__ n_unique_p,
                                   int32_t *__restrict__ rank_of_orig)
{
    const int nu = (int)*n_unique_p;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        const int32_t x = tmax[j];
        int lo = 0, hi = nu;              // first index with unique[idx] >= x
        while (lo < hi) {
            int mid = (lo + hi) >> 1;
            if ((uint32_t)unique[mid] < (uint32_t)x) lo = mid + 1; else hi = mid;
        }
        rank_of_orig[j] = (lo < nu && unique[lo] == x) ? lo : -1;
    }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_gather_table_values(hipStream_t st, const int32_t *table, int K, int S,
                                      int32_t inf_key, int32_t *out_keys)
{
    long long total = (long long)K * K * K * S;
    int grid = (int)((total + 255) / 256);
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(gather_table_values_kernel, dim3(grid), dim3(256), 0, st, table, K, S,
                       inf_key, out_keys);
    return hipGetLastError();
}

// Sorts keys[0][0..n) (clobbering both key buffers), writes the ascending distinct values
// other than drop_key to out_unique and their count to *out_n_unique (device).
hipError_t launch_sort_dedup(hipStream_t st, PrepBuffers &pb, int n, int key_bits,
                             int32_t drop_key, int32_t *out_unique, uint32_t *out_n_unique)
{
    int cur = 0;
    for (int shift = 0; shift < key_bits; shift += 8) {
        hipLaunchKernelGGL(radix_hist_kernel, dim3(SORT_BLOCKS), dim3(WAVE), 0, st,
                           pb.keys[cur], n, shift, pb.hist);
        uint32_t *totals = pb.hist + RADIX * SORT_BLOCKS;
        hipLaunchKernelGGL(digit_scan_kernel, dim3(RADIX), dim3(SORT_BLOCKS), 0, st, pb.hist,
                           totals);
        hipLaunchKernelGGL(digit_base_kernel, dim3(1), dim3(RADIX), 0, st, totals);
        hipLaunchKernelGGL(radix_scatter_kernel, dim3(SORT_BLOCKS), dim3(WAVE), 0, st,
                           pb.keys[cur], pb.keys[cur ^ 1], n, shift, pb.hist, totals);
        cur ^= 1;
    }
    const int nb = (n + DEDUP_TILE - 1) / DEDUP_TILE;
    hipLaunchKernelGGL(dedup_count_kernel, dim3(nb), dim3(1024), 0, st, pb.keys[cur], n, drop_key,
                       pb.block_cnt);
    hipLaunchKernelGGL(scan_u32_kernel, dim3(1), dim3(1024), 0, st, pb.block_cnt, nb,
                       out_n_unique);
    hipLaunchKernelGGL(dedup_write_kernel, dim3(nb), dim3(1024), 0, st, pb.keys[cur], n, drop_key,
                       pb.block_cnt, out_unique);
    return hipGetLastError();
}

// A list of n <= LIST_SORT_MAX values on the device: its ascending distinct values, their number (also to the state), and
// each value's place among them (rank_of_orig may be null)
hipError_t launch_list_sort(hipStream_t st, const int32_t *tmax, int n, int32_t *out_unique, uint32_t *out_n_unique,
                            SolveState *state, int32_t *rank_of_orig)
{
    int N2 = 2;
    while (N2 < n) N2 <<= 1;
    const size_t lds = (size_t)2 * N2 * 4;
    if (lds > 32 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)list_sort_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(list_sort_kernel, dim3(1), dim3(1024), lds, st, tmax, n, N2, out_unique, out_n_unique, state, rank_of_orig);
    return hipGetLastError();
}

hipError_t launch_bitmap_clear(hipStream_t st, uint32_t *work, int32_t max_value)
{
    const int words = max_value / 32 + 1;
    hipLaunchKernelGGL(bitmap_clear_kernel, dim3(std::min((words + 1023) / 1024, 256)), dim3(1024), 0, st, work, words);
    return hipGetLastError();
}

// Ascending distinct finite values of the table's entries with last >= first layer, all known
// to be <= max_value, to out_unique and their count to *out_n_unique.
// `work` holds the bitmap, which is clear, and the block counts: distinct_bitmap_words(max_value) uint32.
hipError_t launch_distinct_by_bitmap(hipStream_t st, const int32_t *table, int K, int S,
                                     int32_t max_value, uint32_t *work, int32_t *out_unique,
                                     uint32_t *out_n_unique)
{
    const int words = max_value / 32 + 1;
    const int nb = (words + 1023) / 1024;
    uint32_t *bm = work, *block_cnt = work + words;
    const int total = K * K * S * ((K + 7) / 8);
    if (max_value < DISTINCT_LOCAL_MAX)
        hipLaunchKernelGGL(bitmap_mark_kernel<true>, dim3(std::min((total + 1023) / 1024, 256)), dim3(1024), (size_t)words * 4,
                           st, table, K, S, words, bm);
    else
        hipLaunchKernelGGL(bitmap_mark_kernel<false>, dim3(std::min((total + 1023) / 1024, 2048)), dim3(1024), 0, st, table, K,
                           S, words, bm);
    const bool few = nb <= 16;
    if (!few) hipLaunchKernelGGL(bitmap_count_kernel, dim3(nb), dim3(1024), 0, st, bm, words, block_cnt);
    hipLaunchKernelGGL(bitmap_write_kernel, dim3(nb), dim3(1024), 0, st, bm, words, block_cnt, few ? 0 : 1, out_unique,
                       out_n_unique);
    return hipGetLastError();
}

size_t distinct_bitmap_words(int32_t max_value)
{
    const size_t words = (size_t)max_value / 32 + 1;
    return words + (words + 1023) / 1024 + 1;
}

hipError_t launch_rank_lookup(hipStream_t st, const int32_t *tmax, int n, const int32_t *unique,
                              const uint32_t *n_unique, int32_t *rank_of_orig)
{
    int grid = (n + 255) / 256;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(rank_lookup_kernel, dim3(grid), dim3(256), 0, st, tmax, n, unique, n_unique,
                       rank_of_orig);
    return hipGetLastError();
}

}  // namespace alpa
