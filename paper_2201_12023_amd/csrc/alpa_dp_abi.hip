// C ABI of libalpa_dp: argument checks, device buffers, and the order in which the
// kernels of one solve are queued.  All arithmetic of the method is in the kernels.
#include "../../include/alpa_dp.h"
#include "internal.hpp"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

using namespace alpa;

static_assert(sizeof(alpa_plan_t) == 2072, "plan layout differs from the kernels' PlanDev");

static thread_local std::string g_err;

static int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

// for the library's other translation units: same thread-local message
extern "C" __attribute__((visibility("hidden"))) int alpa_dp_set_error_(int code, const char *msg)
{
    return fail(code, msg);
}

#define HIPCHK(expr)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(e_ == hipErrorOutOfMemory ? ALPA_DP_ENOMEM : ALPA_DP_EHIP,          \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                 \
    } while (0)

// A group of arrays that grows with the candidate lists.  The arrays it has outgrown stay where they are to
// the end of the handle: a solve that is queued, or recorded into a graph, still uses them, so growing
// neither waits nor releases anything.  The room at least doubles, so what is kept is less than what is in use.
struct GrowingArena {
    void *mem = nullptr;
    int cap = 0;
    void *kept[32] = {};
    int n_kept = 0;
    void release()
    {
        (void)hipFree(mem);
        while (n_kept) (void)hipFree(kept[--n_kept]);
        mem = nullptr;
        cap = 0;
    }
};

struct alpa_dp {
    Problem p{};
    int device = 0;
    hipStream_t stream = nullptr;
    int32_t max_finite = -1;        // largest finite table entry with last >= first layer
    int key_bits_table = 1;
    int n_table_keys = 0;           // K * K(K+1)/2 * S
    int n_distinct = 0;             // distinct finite table values
    int n_cu = 0;
    bool fast_ok = false;
    int KP = 0;
    int fast_grid_max[3] = {0, 0, 0}, generic_grid_max = 0;   // [nc] for nc = 1, 2

    // One allocation per group of arrays (an allocation and its release cost tens of microseconds each):
    // what lives as long as the handle, the keys of the sorts, the per-candidate arrays, and those of a
    // sweep.  The pointers below are parts of these.
    void *arena = nullptr, *sweep_arena = nullptr, *distinct_arena = nullptr;
    GrowingArena keys, cands;
    bool recorded = false;          // a solve has been recorded into a graph
    int32_t *d_table = nullptr, *d_sizes = nullptr, *d_recs = nullptr, *d_gmin = nullptr;
    int32_t *d_bandrecs = nullptr, *d_bandends = nullptr, *d_bandthr = nullptr, *d_backs = nullptr;
    int32_t *d_least = nullptr, *d_front = nullptr, *d_graph = nullptr;
    bool band_ok = false;
    bool sparse_ok = false;         // there is room for candidates to go by graphs (kernels_sparse.hip)
    bool ordered = false;           // and the table's latencies do not fall with the number of stages
    uint16_t *d_kept = nullptr;     // plans of those that are settled
    int32_t *d_kept_from = nullptr;
    BandShape band{};
    BandShapes band_shapes{};
    int32_t *d_bounds = nullptr;    // what the table says about every candidate (launch_table_bounds)
    int32_t *d_no_bounds = nullptr; // the same layout, saying nothing
    int32_t *d_bound_work = nullptr;
    bool have_bounds = false;       // of the present table: computed by the first solve that wants them
    bool have_exact_bounds = false; // better ones for the band kernel, by the second one (launch_band_exact_bounds)
    PrepBuffers pb{};
    int32_t *d_distinct = nullptr;
    uint32_t *d_ncount = nullptr;   // [2]: distinct table values, distinct caller candidates
    int32_t *d_cand = nullptr, *d_rank = nullptr, *d_tmax_stage = nullptr;
    int32_t *d_Fmin = nullptr, *d_Sbest = nullptr, *d_knots = nullptr, *d_list = nullptr, *d_todo = nullptr, *d_slot = nullptr;
    int64_t *d_T = nullptr, *d_outT_stage = nullptr, *d_chunkmin = nullptr;
    SolveState *d_state = nullptr;
    int32_t *d_scratch = nullptr, *d_Fall = nullptr, *d_tmpFS = nullptr;
    alpa_plan_t *d_plan_tmp = nullptr, *d_best_plan = nullptr;
    // sweep over B (allocated on first use, for up to sw_cap values)
    int sw_cap = 0, sw_sets = 1;    // sw_sets: sets of layers in d_sw_Fall
    int32_t *d_sw_B = nullptr, *d_sw_c = nullptr, *d_sw_s = nullptr, *d_sw_FS = nullptr;
    int32_t *d_sw_n = nullptr;      // [chunk][2]: number of B values, ticket of the plan-recovery run
    SolveState *d_sw_state = nullptr;
    int32_t *d_sw_Fall = nullptr;
    alpa_plan_t *d_sw_plans = nullptr;
    int clock_khz = 100000;         // of the clock that kernels read
    bool any_solve = false;
    enum { NOT_TIMED, TIMED, RECORDED } timed = NOT_TIMED;   // the last solve's times are in d_state (a recorded one's are a replay's)
    bool have_best = false;         // d_best_plan holds the best of a solve made with the current
                                    // table and B (sweeps do not touch it)
    // tuning (alpa_dp_set_tuning); 0 = the library's own choice
    int tune_nc = 0, tune_sort = 0, tune_wg_per_cu = 0, tune_grid = 0, tune_no_groups = 0;
    int fast_per_cu[3] = {0, 0, 0};  // resident workgroups per compute unit, [nc]
};

// Parts of one allocation: `layout` names them twice, first to count, then to place them.
struct Carver {
    char *base = nullptr;
    size_t used = 0;
    template <class T> void operator()(T *&p, size_t n)
    {
        p = base ? (T *)(base + used) : nullptr;
        used += (n * sizeof(T) + 255) & ~(size_t)255;
    }
};

// All or nothing: after a failure *arena and every pointer of the layout are null.
template <class Layout>
static int carve(void **arena, Layout layout)
{
    (void)hipFree(*arena);
    *arena = nullptr;
    Carver count;
    layout(count);
    const hipError_t e = hipMalloc(arena, count.used);
    if (e != hipSuccess) (void)hipGetLastError();  // reported here, not to be found by the next launch
    HIPCHK(e);
    Carver place{(char *)*arena};
    layout(place);
    return ALPA_DP_OK;
}

// Work area of the sorts (of the table's values or of a caller's list) for `c` keys; for the values of a
// table it holds a bitmap instead
static void key_layout(alpa_dp *h, size_t c, Carver &take)
{
    take(h->pb.keys[0], c);
    take(h->pb.keys[1], c);
    take(h->pb.block_cnt, c / 4096 + 2);
}

// Per-candidate arrays for `c` candidates
static void candidate_layout(alpa_dp *h, size_t c, Carver &take)
{
    take(h->d_cand, c);
    take(h->d_list, c);
    take(h->d_todo, h->sparse_ok ? c : 0);
    take(h->d_slot, h->sparse_ok ? c : 0);
    take(h->d_rank, c);
    take(h->d_tmax_stage, c);
    take(h->d_Fmin, c + 1);                        // + one spare slot (see FastArgs)
    take(h->d_Sbest, c + 1);
    take(h->d_T, c);
    take(h->d_outT_stage, c);
    take(h->d_chunkmin, c / PRUNE_CHUNK + 2);
}

// Is the handle's stream being recorded into a graph?  (The null stream never is, and asking about it while
// another one is recorded is an error.)
static int stream_is_recorded(const alpa_dp *h, bool *yes)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (h->stream) HIPCHK(hipStreamIsCapturing(h->stream, &status));
    *yes = status != hipStreamCaptureStatusNone;
    return ALPA_DP_OK;
}

typedef void (*ArenaLayout)(alpa_dp *, size_t, Carver &);

static hipError_t new_arrays(alpa_dp *h, GrowingArena &g, int cap, ArenaLayout layout)
{
    Carver count;
    layout(h, (size_t)cap, count);
    void *fresh = nullptr;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;    // an allocation is no part of a recording
    hipError_t e = hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) {
        e = hipMalloc(&fresh, count.used);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (e != hipSuccess) {                         // (the pointers are null now: see grow)
        (void)hipGetLastError();                   // handled by the caller, not to be found by the next launch
        return e;
    }
    Carver place{(char *)fresh};
    layout(h, (size_t)cap, place);
    if (g.mem) g.kept[g.n_kept++] = g.mem;
    g.mem = fresh;
    g.cap = cap;
    return hipSuccess;
}

// Room for `need` entries.  A failure leaves the group as it was; where memory is short and no graph needs the
// outgrown arrays they are released first, and then a failure leaves a capacity of 0, so that the next
// solve tries again.
static int grow(alpa_dp *h, GrowingArena &g, int need, ArenaLayout layout)
{
    if (g.cap >= need) return ALPA_DP_OK;
    bool recorded = false;
    const int rc = stream_is_recorded(h, &recorded);
    if (rc) return rc;
    const int roomy = (int)std::max<long long>(need, std::min<long long>(2ll * g.cap, INT32_MAX - 4096));
    hipError_t e = new_arrays(h, g, roomy, layout);
    if (e == hipErrorOutOfMemory && !recorded && !h->recorded) {
        HIPCHK(hipStreamSynchronize(h->stream));
        g.release();
        e = new_arrays(h, g, need, layout);
    }
    if (e != hipSuccess) {
        Carver back{(char *)g.mem};                // (all null if there is nothing to go back to)
        layout(h, (size_t)g.cap, back);
        return fail(e == hipErrorOutOfMemory ? ALPA_DP_ENOMEM : ALPA_DP_EHIP,
                    std::string("arrays for ") + std::to_string(need) + " candidates: " + hipGetErrorString(e));
    }
    return ALPA_DP_OK;
}

static bool distinct_by_bitmap(const alpa_dp *h)
{
    // (a bitmap of more words than there are keys costs more than the sort's smallest passes)
    return h->max_finite >= 0 && h->max_finite < DISTINCT_BITMAP_MAX && !h->tune_sort &&
           (h->max_finite < DISTINCT_LOCAL_MAX || h->max_finite / 32 < h->n_table_keys);
}

// From the start there is room for lists of ordinary length (both groups together stay below 2 MiB, from where
// on an allocation and its release take longer: room for every entry of the table made a planning call of 32
// layers on 4 x 8 773 instead of 680 us).
constexpr int ORDINARY_LIST = 16384;
static int ordinary_list(const alpa_dp *h) { return std::min(std::max(h->n_table_keys, 1024), ORDINARY_LIST); }

// Keys for a list of n_list and for what finds the table's values: the words of a bitmap, or a key per entry
static int ensure_keys(alpa_dp *h, int n_list)
{
    const int find = distinct_by_bitmap(h) ? (int)distinct_bitmap_words(h->max_finite) : h->n_table_keys;
    return grow(h, h->keys, std::max(std::max(find, n_list), ordinary_list(h)), key_layout);
}

// Everything that a solve needs: keys, and per-candidate arrays for the distinct table values or the caller's list
static int ensure_candidate_arrays(alpa_dp *h, int n_list)
{
    const int rc = ensure_keys(h, n_list);
    if (rc) return rc;
    return grow(h, h->cands, std::max(std::max(h->n_distinct, n_list), ordinary_list(h)), candidate_layout);
}

// one kernel recovers the layers of all winners of a sweep (else a launch per layer, winner by winner)
static bool plan_slabs(const alpa_dp *h) { return h->band_ok || (h->fast_ok && h->p.D <= 64); }

// int32 of one winner's layers, and the winners whose layers are kept at a time: up to 1 GiB of them, as many as there is
// memory for, and at least the one set that the handle has anyway
static size_t slab_ints(const alpa_dp *h) { return (size_t)(h->p.Smax + 1) * (size_t)(h->p.K + 2) * (h->p.D + 1); }
static int sweep_chunk(const alpa_dp *h, int n_B) { return std::min(n_B, h->sw_sets); }

static int alloc_sweep_arrays(alpa_dp *h, int n_B)
{
    const size_t n = (size_t)n_B;
    h->sw_cap = 0;
    size_t sets = plan_slabs(h) ? std::max<size_t>(1, std::min<size_t>(n, (1ull << 28) / slab_ints(h))) : 1;
    for (;; sets /= 2) {
        const int rc = carve(&h->sweep_arena, [&](Carver &take) {
            take(h->d_sw_B, n);
            take(h->d_sw_c, n);
            take(h->d_sw_s, n);
            take(h->d_sw_FS, 2 * (n + 1));
            take(h->d_sw_n, 2 * n);
            take(h->d_sw_state, n);
            take(h->d_sw_plans, n);
            if (sets > 1) take(h->d_sw_Fall, sets * slab_ints(h));
        });
        if (rc == ALPA_DP_ENOMEM && sets > 1) continue;
        if (rc) return rc;
        break;
    }
    if (sets == 1) h->d_sw_Fall = h->d_Fall;
    h->sw_sets = (int)sets;
    h->sw_cap = n_B;
    return ALPA_DP_OK;
}

static int bits_for(uint32_t v)
{
    int b = 1;
    while (b < 32 && (v >> b)) ++b;
    return b;
}

// distinct finite table values -> d_distinct, count -> d_ncount[0]; `cleared`: the bitmap (in the second key buffer)
static int queue_table_candidates(alpa_dp *h, bool cleared = false)
{
    const int rc = ensure_keys(h, 0);
    if (rc) return rc;
    // small values: one bit per value instead of a sort (the second key buffer is the work area)
    if (distinct_by_bitmap(h)) {
        if (!cleared) HIPCHK(launch_bitmap_clear(h->stream, (uint32_t *)h->pb.keys[1], h->max_finite));
        HIPCHK(launch_distinct_by_bitmap(h->stream, h->d_table, h->p.K, h->p.S, h->max_finite,
                                         (uint32_t *)h->pb.keys[1], h->d_distinct,
                                         h->d_ncount + 0));
        return ALPA_DP_OK;
    }
    const int32_t inf_key = h->max_finite + 1;
    HIPCHK(launch_gather_table_values(h->stream, h->d_table, h->p.K, h->p.S, inf_key,
                                      h->pb.keys[0]));
    HIPCHK(launch_sort_dedup(h->stream, h->pb, h->n_table_keys, h->key_bits_table, inf_key,
                             h->d_distinct, h->d_ncount + 0));
    return ALPA_DP_OK;
}

// the table as the band kernel and what it takes beforehand read it
static hipError_t launch_band_table(alpa_dp *h)
{
    const hipError_t e = launch_repack_band(h->stream, h->d_table, h->p, h->band_shapes, h->d_bandrecs, h->d_bandends, h->d_bounds, !h->ordered);
    return e != hipSuccess ? e : launch_front_table(h->stream, h->d_table, h->band_shapes, h->p, h->d_least, h->d_front);
}

// what the table says about every candidate -> d_bounds; `recorded`: a graph's replays behind the first find the band
// kernel's bounds there, and only look (46 us at 24 layers on 2 x 8, 165 at 64 on 8 x 8, 550 at 48 on 32 x 8 each otherwise)
static int queue_bounds(alpa_dp *h, bool recorded)
{
    if (h->band_ok)
        HIPCHK(launch_band_bounds(h->stream, h->d_table, h->band_shapes, h->p, h->max_finite,
                                  BandWork{h->d_least, h->d_front, h->d_bandthr, h->d_backs, h->d_graph},
                                  h->d_bounds, recorded));
    else
        HIPCHK(launch_table_bounds(h->stream, h->p, h->d_table, h->d_sizes, h->d_bound_work, h->d_bounds));
    return ALPA_DP_OK;
}

// better ones, for tables that want them (launch_band_exact_bounds)
static int queue_exact_bounds(alpa_dp *h, bool recorded)
{
    HIPCHK(launch_band_exact_bounds(h->stream, h->band_shapes, h->band, h->p, h->max_finite, h->d_bandrecs, h->d_bandends,
                                    h->d_bound_work, h->d_bandthr, h->d_bounds, recorded));
    return ALPA_DP_OK;
}

extern "C" const char *alpa_dp_last_error(void) { return g_err.c_str(); }

extern "C" void alpa_dp_destroy(alpa_dp_t *h)
{
    if (!h) return;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(h->device);
    (void)hipStreamSynchronize(h->stream);
    (void)hipFree(h->arena); (void)hipFree(h->sweep_arena); (void)hipFree(h->distinct_arena);
    h->keys.release();
    h->cands.release();
    (void)hipSetDevice(prev);
    delete h;
}

// Argument checks common to both ways of creating a handle; fills sizes[q] = n_q * m_q.
static int check_problem(int K, int N, int M, int B, const alpa_shape_t *shapes, int num_shapes,
                         std::vector<int32_t> &sizes)
{
    if (!shapes) return fail(ALPA_DP_EINVAL, "shapes is null");
    if (K < 1 || K > ALPA_DP_MAX_K) return fail(ALPA_DP_EINVAL, "K out of range");
    if (N < 1 || M < 1 || (long long)N * M > ALPA_DP_MAX_DEVICES)
        return fail(ALPA_DP_EINVAL, "N x M out of range");
    if ((M & (M - 1)) != 0) return fail(ALPA_DP_EINVAL, "M must be a power of two");
    if (B < 1) return fail(ALPA_DP_EINVAL, "B must be >= 1");
    if (num_shapes < 1 || num_shapes > ALPA_DP_MAX_SHAPES)
        return fail(ALPA_DP_EINVAL, "num_shapes out of range");
    sizes.resize(num_shapes);
    for (int q = 0; q < num_shapes; ++q) {
        const int n = shapes[q].n, m = shapes[q].m;
        const bool one_d = n == 1 && m >= 1 && m <= M && (m & (m - 1)) == 0;
        const bool two_d = m == M && n >= 2 && n <= N;
        if (!one_d && !two_d) return fail(ALPA_DP_EINVAL, "shape outside the submesh family");
        sizes[q] = n * m;
    }
    return ALPA_DP_OK;
}

// Device side of handle creation.  `fill_table` puts the table into h->d_table (already
// allocated) and sets h->max_finite; everything else follows from those two.
template <class FillTable>
static int create_on_device(alpa_dp *h, const std::vector<int32_t> &sizes, FillTable fill_table)
{
    const int K = h->p.K, S = h->p.S, D = h->p.D;
    HIPCHK(hipGetDevice(&h->device));
    HIPCHK(hipDeviceGetAttribute(&h->n_cu, hipDeviceAttributeMultiprocessorCount, h->device));
    HIPCHK(hipDeviceGetAttribute(&h->clock_khz, hipDeviceAttributeWallClockRate, h->device));
    const size_t LS = (size_t)(K + 2) * (D + 1);
    // general kernel: two F layers per resident workgroup, at most 256 MiB in total
    int gg = h->n_cu * 4;
    while (gg > 1 && (size_t)gg * 2 * LS * 4 > (256ull << 20)) gg /= 2;
    h->generic_grid_max = gg;
    // The band kernel, a workgroup per candidate, wherever its layers fit in LDS (up to 243 layers on 8 x 8, 123 on
    // 16 x 8, 59 on 32 x 8).  On small meshes most lanes of its waves have nothing to do, and the register/LDS kernel takes
    // several candidates to a wave.  What the band kernel wants to know of a table (band_thresholds_kernel) costs a first
    // solve more than it saves there, so that one stays on up to 4 devices (us, first solve and later ones: 128 layers on 1 x 4,
    // 1000 candidates: 241 and 212 against 321 and 199) and on up to 8 with up to 64 layers (64 on 1 x 8,
    // 2048: 252 and 215 against 298 and 190; but 72 on 2 x 4, 2048: 288 and 241 against 280 and 195).  It also takes
    // what is left of 65 to 128 devices (two windows: from 89 layers on), the general kernel the rest.
    const bool groups_serve = K <= 128 && (D <= 4 || (D <= 8 && K <= 64));
    // (shapes of one device count, i.e. repeated ones, are one shape to it)
    std::vector<int32_t> band_sizes, first, next(S, -1), last;
    for (int q = 0; q < S; ++q) {
        const int x = (int)(std::find(band_sizes.begin(), band_sizes.end(), sizes[q]) - band_sizes.begin());
        if (x == (int)band_sizes.size()) {
            band_sizes.push_back(sizes[q]);
            first.push_back(q);
            last.push_back(q);
        } else {
            next[last[x]] = q;
            last[x] = q;
        }
    }
    const int SB = (int)band_sizes.size();
    h->band = band_shape(K, D, SB, band_sizes.data());
    h->band_ok = !groups_serve && h->band.nbuf != 0;
    h->sparse_ok = h->band_ok && SB == S;          // (of shapes with equal device counts the graph would not know the lowest)
    h->fast_ok = !h->band_ok && K <= 128 && (D <= 8 || (D > WAVE && D <= 128 && K > 16 * (FAST_WIDE_NWK - 1)));
    int rc = carve(&h->arena, [&](Carver &take) {
        take(h->d_table, (size_t)K * K * K * S);
        take(h->d_sizes, S + table_bounds_ints(h->p) + 2 * SB + S);    // behind them d_no_bounds and band_shapes
        take(h->pb.hist, SORT_RADIX * SORT_SLICES + SORT_RADIX);   // counts + totals
        take(h->d_ncount, 2);
        take(h->d_state, 1);
        take(h->d_tmpFS, 4);
        take(h->d_knots, 2 * REFINE_MAX_KNOTS);
        take(h->d_plan_tmp, 1);
        take(h->d_best_plan, 1);
        take(h->d_Fall, (size_t)(h->p.Smax + 1) * LS);
        take(h->d_bounds, table_bounds_ints(h->p) + (h->band_ok ? BAND_TOTALS : 0));
        take(h->d_bound_work, h->band_ok ? 2 * (size_t)h->p.Smax : table_bounds_work(h->p));
        take(h->d_scratch, (size_t)gg * 2 * LS);
        if (h->band_ok) {
            take(h->d_bandrecs, band_table_ints(K, h->p.Smax, SB));
            take(h->d_bandends, band_ends_ints(K, h->p.Smax, SB));
            take(h->d_bandthr, band_thresholds_ints(K, D));
            take(h->d_backs, band_thresholds_ints(K, D));
            take(h->d_least, front_least_ints(K, SB));
            take(h->d_front, front_table_ints(K, SB));
            if (h->sparse_ok) {
                take(h->d_graph, graph_table_ints(K, D));
                take(h->d_kept, (size_t)SPARSE_PLANS * K);
                take(h->d_kept_from, SPARSE_PLANS);
            }
        }
        if (h->fast_ok) {
            take(h->d_recs, fast_table_ints(K, S));
            take(h->d_gmin, fast_group_min_ints(K, D, S));
        }
    });
    if (rc) return rc;
    rc = fill_table();
    if (rc) return rc;
    if (h->max_finite >= 0 && (long long)K * h->max_finite >= (1ll << 30))
        return fail(ALPA_DP_EOVERFLOW, "K * largest finite latency >= 2^30");
    h->key_bits_table = bits_for((uint32_t)(h->max_finite + 1));
    h->n_table_keys = K * (K * (K + 1) / 2) * S;
    // (the call ends with a synchronisation: `up` may go away after the return)
    std::vector<int32_t> up(sizes);
    up.insert(up.end(), table_bounds_ints(h->p), -1);
    up[S + h->p.Smax + 1] = 0;                     // any t_max may have a plan, of an unknown number of stages
    up[S + h->p.Smax + 3] = DEV_INF;
    h->d_no_bounds = h->d_sizes + S;
    const int32_t *shapes_at = h->d_sizes + up.size();
    up.insert(up.end(), band_sizes.begin(), band_sizes.end());
    up.insert(up.end(), first.begin(), first.end());
    up.insert(up.end(), next.begin(), next.end());
    h->band_shapes = BandShapes{SB, S, shapes_at, SB < S ? shapes_at + SB : nullptr, shapes_at + 2 * SB};
    HIPCHK(hipMemcpyAsync(h->d_sizes, up.data(), up.size() * 4, hipMemcpyHostToDevice, h->stream));
    HIPCHK(hipMemsetAsync(h->d_state, 0, sizeof(SolveState), h->stream));
    HIPCHK(launch_init_best_plan(h->stream, h->d_best_plan));
    if (h->band_ok) HIPCHK(launch_band_table(h));
    if (h->fast_ok) {
        h->KP = 16 * ((K + 15) / 16);
        HIPCHK(launch_repack_fast(h->stream, h->d_table, K, D, S, h->KP, h->d_recs, h->d_gmin));
        for (int nc = 1; nc <= 2; ++nc) {
            int per_cu = fast_kernel_blocks_per_cu(K, nc);
            if (per_cu < 1) return fail(ALPA_DP_EHIP, "fast kernel does not fit on a CU");
            h->fast_per_cu[nc] = per_cu;
            h->fast_grid_max[nc] = h->n_cu * per_cu;
        }
    }
    int rc2 = carve(&h->distinct_arena, [&](Carver &take) {
        take(h->d_distinct, (size_t)std::min<long long>(h->n_table_keys, (long long)h->max_finite + 2));
    });
    if (rc2) return rc2;
    // length of the full candidate list
    rc2 = queue_table_candidates(h);
    if (rc2) return rc2;
    uint32_t nd = 0;
    HIPCHK(hipMemcpyAsync(&nd, h->d_ncount, 4, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    h->n_distinct = (int)nd;
    return ensure_candidate_arrays(h, 0);
}

template <class FillTable>
static int create_handle(alpa_dp_t **out, int K, int N, int M, int B,
                         const std::vector<int32_t> &sizes, FillTable fill_table_for)
{
    alpa_dp *h = new (std::nothrow) alpa_dp();
    if (!h) return fail(ALPA_DP_ENOMEM, "host allocation failed");
    const int D = N * M;
    h->p = Problem{K, N, M, D, (int)sizes.size(), std::min(K, D), B};
    const int rc = create_on_device(h, sizes, [&]() { return fill_table_for(h); });
    if (rc != ALPA_DP_OK) {
        std::string keep = g_err;
        alpa_dp_destroy(h);
        g_err = keep;
        return rc;
    }
    *out = h;
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_create(alpa_dp_t **out, const int32_t *cost_table, int K, int N, int M,
                              int B, const alpa_shape_t *shapes, int num_shapes)
{
    if (!out) return fail(ALPA_DP_EINVAL, "out is null");
    *out = nullptr;
    if (!cost_table || !shapes) return fail(ALPA_DP_EINVAL, "cost_table or shapes is null");
    std::vector<int32_t> sizes;
    int rc = check_problem(K, N, M, B, shapes, num_shapes, sizes);
    if (rc) return rc;
    const int S = num_shapes;
    return create_handle(out, K, N, M, B, sizes, [&](alpa_dp *h) -> int {
        // the range check of the used part of the table (no negative latency; largest finite
        // entry for the overflow proof) is a reduction on the device copy
        int32_t *d_range = h->d_tmpFS;             // (three; free until the first solve)
        HIPCHK(hipMemcpyAsync(h->d_table, cost_table, (size_t)K * K * K * S * 4,
                              hipMemcpyHostToDevice, h->stream));
        HIPCHK(launch_table_range(h->stream, h->d_table, K, S, h->p.Smax, d_range));
        int32_t range[3] = {0, -1, 1};
        HIPCHK(hipMemcpyAsync(range, d_range, sizeof(range), hipMemcpyDeviceToHost, h->stream));
        HIPCHK(hipStreamSynchronize(h->stream));
        if (range[0] < 0) return fail(ALPA_DP_EINVAL, "negative latency in cost_table");
        h->max_finite = range[1];
        h->ordered = range[2] == 0;
        return ALPA_DP_OK;
    });
}

extern "C" int alpa_dp_create_from_profiles(alpa_dp_t **out, const int32_t *t_l,
                                            const int64_t *mem_stage, const int64_t *mem_act,
                                            int num_options, int64_t mem_device, int K, int N,
                                            int M, int B, const alpa_shape_t *shapes,
                                            int num_shapes)
{
    if (!out) return fail(ALPA_DP_EINVAL, "out is null");
    *out = nullptr;
    if (!t_l || !mem_stage || !mem_act) return fail(ALPA_DP_EINVAL, "a profile array is null");
    if (num_options < 1 || num_options > ALPA_DP_MAX_OPTIONS)
        return fail(ALPA_DP_EINVAL, "num_options out of range");
    if (mem_device < 0) return fail(ALPA_DP_EINVAL, "mem_device is negative");
    std::vector<int32_t> sizes;
    int rc = check_problem(K, N, M, B, shapes, num_shapes, sizes);
    if (rc) return rc;
    const int S = num_shapes, O = num_options;
    // s * mem_act stays far inside int64 when every figure is below 2^52 (s <= 256)
    for (int k = 0; k < K; ++k)
        for (int i = k; i < K; ++i) {
            const size_t e0 = ((size_t)k * K + i) * S * O, cnt = (size_t)S * O;
            for (size_t x = e0; x < e0 + cnt; ++x) {
                if (t_l[x] < 0) return fail(ALPA_DP_EINVAL, "negative latency in t_l");
                if (mem_stage[x] < 0 || mem_act[x] < 0 || mem_stage[x] >= (1ll << 52) ||
                    mem_act[x] >= (1ll << 52))
                    return fail(ALPA_DP_EINVAL, "memory figure outside [0, 2^52)");
            }
        }
    if (mem_device >= (1ll << 62)) return fail(ALPA_DP_EINVAL, "mem_device too large");
    return create_handle(out, K, N, M, B, sizes, [&](alpa_dp *h) -> int {
        const size_t n = (size_t)K * K * S * O;
        void *inputs = nullptr;
        int32_t *d_t = nullptr, *d_max = h->d_tmpFS;    // (free until the first solve)
        int64_t *d_ms = nullptr, *d_ma = nullptr;
        auto body = [&]() -> int {
            const int rc1 = carve(&inputs, [&](Carver &take) { take(d_t, n); take(d_ms, n); take(d_ma, n); });
            if (rc1) return rc1;
            HIPCHK(hipMemcpyAsync(d_t, t_l, n * 4, hipMemcpyHostToDevice, h->stream));
            HIPCHK(hipMemcpyAsync(d_ms, mem_stage, n * 8, hipMemcpyHostToDevice, h->stream));
            HIPCHK(hipMemcpyAsync(d_ma, mem_act, n * 8, hipMemcpyHostToDevice, h->stream));
            HIPCHK(launch_build_table(h->stream, d_t, d_ms, d_ma, K, S, O, mem_device, h->d_table,
                                      d_max));
            int32_t mx = -1;
            HIPCHK(hipMemcpyAsync(&mx, d_max, 4, hipMemcpyDeviceToHost, h->stream));
            HIPCHK(hipStreamSynchronize(h->stream));
            h->max_finite = mx;
            h->ordered = true;                     // (what fits with more stages fits with fewer)
            return ALPA_DP_OK;
        };
        const int rc2 = body();
        (void)hipFree(inputs);
        return rc2;
    });
}

extern "C" int alpa_dp_restrict_equal_layers(alpa_dp_t *h)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    const int K = h->p.K, D = h->p.D, S = h->p.S;
    HIPCHK(launch_equal_layer_mask(h->stream, h->d_table, K, S));
    h->ordered = false;
    if (h->band_ok) HIPCHK(launch_band_table(h));
    if (h->fast_ok) {
        HIPCHK(launch_repack_fast(h->stream, h->d_table, K, D, S, h->KP, h->d_recs, h->d_gmin));
    }
    // (a graph recorded after the first solve reads the bounds and does not compute them)
    if (h->have_bounds) {
        int rcb = queue_bounds(h, false);
        if (!rcb && h->have_exact_bounds) rcb = queue_exact_bounds(h, false);
        if (rcb) return rcb;
    }
    // the candidate list changes with the table; the running best belonged to the old one
    int rc = queue_table_candidates(h);
    if (rc) return rc;
    uint32_t nd = 0;
    HIPCHK(hipMemcpyAsync(&nd, h->d_ncount, 4, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(launch_init_best_plan(h->stream, h->d_best_plan));
    HIPCHK(hipStreamSynchronize(h->stream));
    h->n_distinct = (int)nd;
    h->any_solve = false;
    h->have_best = false;
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_get_table(alpa_dp_t *h, int32_t *out_table)
{
    if (!h || !out_table) return fail(ALPA_DP_EINVAL, "null argument");
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    const size_t bytes = (size_t)h->p.K * h->p.K * h->p.K * h->p.S * 4;
    HIPCHK(hipMemcpyAsync(out_table, h->d_table, bytes, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_set_stream(alpa_dp_t *h, void *hip_stream)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    HIPCHK(hipStreamSynchronize(h->stream));
    h->stream = (hipStream_t)hip_stream;
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_set_B(alpa_dp_t *h, int B)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    if (B < 1) return fail(ALPA_DP_EINVAL, "B must be >= 1");
    if (B == h->p.B) return ALPA_DP_OK;
    // T* of Eq. 4 under different B values do not compare: the running best starts over
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    HIPCHK(launch_init_best_plan(h->stream, h->d_best_plan));
    h->have_best = false;
    h->p.B = B;
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_set_tuning(alpa_dp_t *h, int key, int value)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    switch (key) {
    case ALPA_DP_TUNE_CANDIDATES_PER_WG:
        if (value < 0 || value > 2) return fail(ALPA_DP_EINVAL, "candidates per workgroup: 0, 1 or 2");
        h->tune_nc = value;
        return ALPA_DP_OK;
    case ALPA_DP_TUNE_DISTINCT_BY_SORT:
        if (value < 0 || value > 1) return fail(ALPA_DP_EINVAL, "distinct values by sort: 0 or 1");
        h->tune_sort = value;
        return ALPA_DP_OK;
    case ALPA_DP_TUNE_WG_PER_CU:
        if (value < 0) return fail(ALPA_DP_EINVAL, "workgroups per compute unit: >= 0");
        h->tune_wg_per_cu = value;
        for (int nc = 1; nc <= 2; ++nc) {
            const int per_cu = (value >= 1 && value < h->fast_per_cu[nc]) ? value : h->fast_per_cu[nc];
            h->fast_grid_max[nc] = h->n_cu * per_cu;
        }
        return ALPA_DP_OK;
    case ALPA_DP_TUNE_LANE_GROUPS:
        if (value < 0 || value > 64 || (value & (value - 1)) != 0)
            return fail(ALPA_DP_EINVAL, "lane groups: 0 (own choice), 1 (off) or 2, 4, .. 64 groups");
        h->tune_no_groups = value;
        return ALPA_DP_OK;
    case ALPA_DP_TUNE_WORKGROUPS:
        if (value < 0) return fail(ALPA_DP_EINVAL, "workgroups: >= 0");
        h->tune_grid = value;
        return ALPA_DP_OK;
    default:
        return fail(ALPA_DP_EINVAL, "unknown tuning key");
    }
}

extern "C" int alpa_dp_count_candidates(alpa_dp_t *h, int *out_n)
{
    if (!h || !out_n) return fail(ALPA_DP_EINVAL, "null argument");
    *out_n = h->n_distinct;
    return ALPA_DP_OK;
}

// Upper bound, known on the host, of the number of distinct candidates of a solve.
static int candidate_bound(const alpa_dp *h, bool have_list, int n_tmax)
{
    if (have_list) return n_tmax;
    if (n_tmax == 0) return h->n_distinct;
    return std::min(h->n_distinct, n_tmax);
}

// How a list of at most `bound` candidates is evaluated.  Up to `all` candidates worth searching go in one
// round: rounds wait for each other, and a round of the register/LDS kernel takes about as long for 256
// candidates as for 2048 (64 layers on 1 x 8 in lane groups).  Where every candidate keeps a compute unit busy by itself
// (the band kernel) the work counts from fewer on (us in one round and in two: 64 layers on 16 x 8, 1024
// candidates: 2235 and 1367; 48 on 8 x 8, 2048: 716 and 337; but 24 on 2 x 8, 1500: 175 and 177).
// Where a candidate is a wave's pass over a graph, 3072 run at a time and 4096 take little longer than 256 (64 layers on 8 x 8: 66 and
// 28 us, two rounds about 72; 47 on 7 x 8 110 for 4096, 55 for 2048), beyond that half of them are knots.
// Without the bounds the problem is small and one round takes everything.
static RefineBuffers plan_rounds(const alpa_dp *h, int bound, bool one_per_cu, bool with_bounds, bool sparse)
{
    RefineBuffers rb{};
    rb.knots[0] = h->d_knots;
    rb.knots[1] = h->d_knots + REFINE_MAX_KNOTS;
    rb.list = h->d_list;
    rb.all = !with_bounds ? INT32_MAX : sparse ? 4096 : one_per_cu ? 512 : 2048;
    rb.first_round = sparse ? 2048 : 256;          // a candidate per compute unit, or eight
    rb.budget = 512;
    rb.rounds = bound <= rb.all ? 1 : sparse || bound <= 8192 ? 2 : 3;
    return rb;
}

// Does a solve of at most `bound` candidates use the table's bounds?  The band kernel lives on them (and gets better ones with
// the second solve, where the table wants them: band_exact_bounds_kernel).  For the
// others they cost the first solve that does a launch per stage count (3.3 to 6 us each), and save what is left out of the
// recurrence, on every solve.  A small problem's first solve goes without (us before there were bounds, with them, without):
//   12 layers on 1 x 8, all 475    105, 108,  97         48 on 1 x 2, all 2705    102, 115, 109
// and not where they pay at once (40 on 1 x 8, all 5050: 194, 163, 185).  A table that is solved again is worth them:
// 12 layers on 1 x 8 then take 84 us.  A recorded solve would compute them on every replay.
static bool wants_bounds(const alpa_dp *h, int bound, bool recorded)
{
    if (h->have_bounds || (h->any_solve && !recorded) || h->band_ok) return true;
    const int K = h->p.K, D = h->p.D;
    const int most_layers = D <= 2 ? 64 : D <= 8 ? 40 : 0;
    const double work = (double)bound * K * K * h->p.S * D;    // about ten per cell-update and stage count
    return K > most_layers || work >= 8e7;
}

// n_B > 0: sweep over the B values in d_sw_B (Eq. 4 and the selection once per value, plans
// to d_sw_plans); otherwise one solve with the handle's B.
static int solve_dev_impl(alpa_dp *h, const int32_t *d_tmax, int n_tmax, unsigned flags,
                          int64_t *d_out_T, alpa_plan_t *d_out_plan, int key_bits, int n_B = 0)
{
    const Problem &p = h->p;
    const bool have_list = d_tmax != nullptr;
    if (n_tmax < 0) return fail(ALPA_DP_EINVAL, "n_tmax < 0");
    if (have_list && n_tmax == 0) return fail(ALPA_DP_EINVAL, "empty candidate list");
    if (!have_list && n_tmax == 1) return fail(ALPA_DP_EINVAL, "fewer than two quantiles");
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    bool recorded = false;
    {
        int rc = ensure_candidate_arrays(h, have_list ? n_tmax : 0);
        if (!rc) rc = stream_is_recorded(h, &recorded);
        if (rc) return rc;
    }
    if (recorded) h->recorded = true;
    const int bound = candidate_bound(h, have_list, n_tmax);
    const int prune_sel = (flags & ALPA_DP_PRUNE) ? 1 : 0;
    // Skipping a candidate while the recurrence runs is decided with one B; a sweep
    // evaluates every candidate and applies the early-exit rule per B in the selection.
    const int prune = n_B > 0 ? 0 : prune_sel;
    hipStream_t st = h->stream;

    const bool fast = h->fast_ok && !(flags & ALPA_DP_GENERIC);
    const bool band = h->band_ok && !(flags & ALPA_DP_GENERIC);
    const bool sparse = band && h->sparse_ok && h->ordered;
    const SparseOut sparse_out{h->d_todo, &h->d_state->n_todo, h->d_slot, &h->d_state->n_slots, h->d_kept, h->d_kept_from, h->d_state->routes};
    const KeptPlans kept{sparse ? h->d_slot : nullptr, h->d_kept, h->d_kept_from, sparse ? graph_stages(h->d_graph, p.K, p.D) : nullptr};
    Problem p_band = p;
    p_band.S = h->band_shapes.S;
    const bool with_bounds = wants_bounds(h, bound, recorded);
    const RefineBuffers rb = plan_rounds(h, bound, !fast, with_bounds, sparse);
    const int32_t *bounds = with_bounds ? h->d_bounds : h->d_no_bounds;
    // per-candidate results are wanted from every interval; a plan alone from few of them
    const RefineQuery rq{n_B > 0 ? h->d_sw_B : nullptr, p.B, std::max(n_B, 1), prune,
                         (n_B > 0 || !d_out_T) ? 1 : 0, bounds, p.Smax, prune_sel,
                         h->band_ok ? bounds + table_bounds_ints(p) : nullptr, h->max_finite,
                         sparse && rb.rounds > 1 ? graph_heads(h->d_graph, p.K, p.D) : nullptr};
    const bool bitmap = !have_list && distinct_by_bitmap(h);
    HIPCHK(launch_init_state(st, h->d_state, h->d_chunkmin, bound / PRUNE_CHUNK + 1, (uint32_t *)h->pb.keys[1],
                             bitmap ? h->max_finite / 32 + 1 : 0));
    PickQuery pick{};
    if (have_list && n_tmax <= LIST_SORT_MAX) {
        HIPCHK(launch_list_sort(st, d_tmax, n_tmax, h->d_cand, h->d_ncount + 1, h->d_state, d_out_T ? h->d_rank : nullptr));
    } else if (have_list) {
        HIPCHK(hipMemcpyAsync(h->pb.keys[0], d_tmax, (size_t)n_tmax * 4, hipMemcpyDeviceToDevice,
                              st));
        HIPCHK(launch_sort_dedup(st, h->pb, n_tmax, key_bits, /*drop_key=*/-1, h->d_cand,
                                 h->d_ncount + 1));
        HIPCHK(launch_set_candidates(st, h->d_ncount + 1, h->d_state));
        if (d_out_T)
            HIPCHK(launch_rank_lookup(st, d_tmax, n_tmax, h->d_cand, h->d_ncount + 1, h->d_rank));
    } else {
        int rc = queue_table_candidates(h, bitmap);
        if (rc) return rc;
        pick = PickQuery{h->d_distinct, h->d_ncount + 0, n_tmax, h->cands.cap};
        HIPCHK(launch_pick_candidates(st, pick, bound, h->d_cand, h->d_state));
    }
    if (with_bounds && !h->have_bounds) {
        int rc = queue_bounds(h, recorded);
        if (!rc && h->band_ok && recorded) rc = queue_exact_bounds(h, recorded);
        if (rc) return rc;
        h->have_bounds = !recorded;                // (recorded, they are there only after the graph's replay)
    } else if (h->band_ok && !h->have_exact_bounds) {
        const int rc = queue_exact_bounds(h, recorded);
        if (rc) return rc;
        h->have_exact_bounds = !recorded;
    }
    HIPCHK(launch_refine_begin(st, rq, pick, h->d_cand, h->d_state, rb));
    for (int round = 1; bound > 0 && round <= rb.rounds; ++round) {
        const bool last = round == rb.rounds;
        if (round > 1)
            HIPCHK(launch_refine(st, rq, h->d_cand, h->d_Fmin, h->d_state, round - 1, last, rb));
        // candidates of a round before the last are knots: none of them may be skipped
        const int skip = last ? prune : 0;
        if (band) {
            FastArgs fa{p_band, nullptr, h->band_shapes.sizes, h->d_cand, rb.list, &h->d_state->n_list, 0, INT32_MAX,
                        &h->d_state->ticket, &h->d_state->wave_relax, h->d_chunkmin, skip,
                        /*descending=*/prune ? 0 : 1, h->d_Fmin, h->d_Sbest, h->cands.cap, nullptr, nullptr,
                        nullptr, bounds};
            if (sparse) {                          // what is not settled there is left to the recurrence
                HIPCHK(launch_sparse_eval(st, fa, h->d_table, h->d_graph, h->max_finite, sparse_out, (flags & ALPA_DP_COUNT_WORK) != 0,
                                          bound, h->n_cu));
                fa.list = h->d_todo;
                fa.n_list_p = &h->d_state->n_todo;
                fa.ticket = &h->d_state->todo_ticket;
                fa.whole = rb.list;
                fa.n_whole_p = &h->d_state->n_list;
                fa.rest = h->d_todo;               // (not read in a launch that lists what is left itself)
                fa.thin = h->d_state->thin;
                fa.leave_out = last && rq.plan_only;
                fa.B_vals = rq.B_vals;
                fa.n_B = rq.n_B;
            }
            HIPCHK(launch_recurrence_band(st, fa, h->band, h->d_bandrecs, h->d_bandends, h->d_bandthr, h->max_finite,
                                          (flags & ALPA_DP_COUNT_WORK) ? FAST_MODE_COUNT : FAST_MODE_BATCH,
                                          std::max(1, std::min(bound, h->n_cu))));
        } else if (fast) {
            // One candidate per workgroup: eight waves per SIMD and two columns folded into one
            // three-operand minimum, which is faster than two candidates sharing their scalar
            // loads and lanes at four waves per SIMD; the two-candidate form stays available through the
            // tuning call.
            int nc = 1;
            if (h->tune_nc) nc = h->tune_nc;
            const bool wide = p.D > 64;            // two windows of device counts, one candidate
            if (wide) nc = 2;
            // Small meshes: groups of lanes, each with a candidate of its own: as many groups as
            // the mesh allows (less work in total, and fewer, lonelier workgroups, which on these
            // small problems matters as much).  Not for lists so short that every candidate gets a compute unit
            // of its own anyway.
            int group_dp = 0;
            if (nc == 1 && h->tune_no_groups != 1 &&
                (bound > h->n_cu || h->tune_no_groups >= 2)) {
                group_dp = fast_lane_group_width(p.D);
                if (h->tune_no_groups >= 2) group_dp = std::max(group_dp, WAVE / h->tune_no_groups);
            }
            const bool grouped = group_dp != 0;
            const int per_wg = wide ? 1 : (grouped ? WAVE / group_dp : nc);
            const int n_groups = (bound + per_wg - 1) / per_wg;
            const int grid = std::max(
                1, std::min(n_groups, h->tune_grid ? h->tune_grid : h->fast_grid_max[nc]));
            FastArgs fa{p, h->d_recs, h->d_sizes, h->d_cand, rb.list,
                        &h->d_state->n_list, 0, INT32_MAX,
                        &h->d_state->ticket, &h->d_state->wave_relax, h->d_chunkmin, skip,
                        /*descending=*/prune ? 0 : 1, h->d_Fmin, h->d_Sbest, h->cands.cap, nullptr, nullptr, h->d_gmin, bounds};
            fa.grouped = group_dp;
            // Short lists go to a form with more waves per candidate (up to 1024 threads), up to two candidates per
            // compute unit, on 65..128 devices, at half the occupancy, up to one (64 layers on 16 x 8: 257
            // against 536 us, but 760 against 714 for 1024).  How long a list is only the device knows:
            // each launch does nothing unless the list is in its share.  What is beyond goes to the lane groups (1024
            // candidates, recurrence alone: 24 layers on 1 x 4 10 us, 27 in a form of eight waves a candidate; 48 on
            // 1 x 8 11 and 30, 40 on 1 x 8 63 and 54).
            const int most = last ? bound : std::max(rb.budget, round == 1 ? rb.all : 0);
            const bool own_form = h->tune_nc || h->tune_no_groups >= 2 || h->tune_grid || h->tune_wg_per_cu;
            if (!(flags & ALPA_DP_COUNT_WORK) && !own_form) {
                fa.n_hi = wide ? h->n_cu : 2 * h->n_cu;
                HIPCHK(launch_recurrence_fast(st, fa, FAST_MODE_FEW, nc, std::min(bound, fa.n_hi)));
                fa.n_lo = fa.n_hi;
                fa.n_hi = INT32_MAX;
            }
            const int form = (flags & ALPA_DP_COUNT_WORK) ? FAST_MODE_COUNT : FAST_MODE_BATCH;
            if (most > fa.n_lo) HIPCHK(launch_recurrence_fast(st, fa, form, nc, grid));
        } else {
            const int grid = std::max(1, std::min(bound, h->generic_grid_max));
            HIPCHK(launch_recurrence_generic(st, p, h->d_table, h->d_sizes, h->d_cand,
                                             rb.list, &h->d_state->n_list, &h->d_state->ticket,
                                             h->d_chunkmin, skip, h->d_Fmin, h->d_Sbest,
                                             h->d_scratch, 2, bounds, grid));
        }
    }
    if (n_B > 0) {
        HIPCHK(launch_sweep_epilogue(st, h->d_sw_B, n_B, h->d_state, h->d_cand, h->d_Fmin,
                                     h->d_Sbest, h->d_sw_state, prune_sel, h->d_sw_c, h->d_sw_s, p, kept, h->d_sw_plans));
        if (plan_slabs(h) && !(flags & ALPA_DP_GENERIC)) {
            const int chunk = sweep_chunk(h, n_B);
            for (int b = 0, x = 0; b < n_B; b += chunk, ++x) {
                const int n = std::min(chunk, n_B - b);
                FastArgs fa{band ? p_band : p, h->d_recs, band ? h->band_shapes.sizes : h->d_sizes, h->d_sw_c + b, nullptr, h->d_sw_n + 2 * x, 0, INT32_MAX,
                            h->d_sw_n + 2 * x + 1,
                            &h->d_state->wave_relax, nullptr, 0, 0, h->d_sw_FS,
                            h->d_sw_FS + (n_B + 1), n_B, h->d_sw_Fall, h->d_sw_s + b, h->d_gmin, bounds};
                if (band)
                    HIPCHK(launch_recurrence_band(st, fa, h->band, h->d_bandrecs, h->d_bandends, h->d_bandthr, h->max_finite,
                                                  FAST_MODE_PLAN, std::min(n, h->n_cu)));
                else
                    HIPCHK(launch_recurrence_fast(st, fa, FAST_MODE_PLAN, 1, std::min(n, h->n_cu)));
                HIPCHK(launch_plan_walk_many(st, p, h->d_table, h->d_sizes, h->d_state, h->d_sw_state + b,
                                             h->d_sw_Fall, slab_ints(h), h->d_sw_plans + b, n));
            }
        } else {
            for (int b = 0; b < n_B; ++b) {        // one slab of layers, reused in stream order
                SolveState *sb = h->d_sw_state + b;
                HIPCHK(launch_plan_layers(st, p, h->d_table, h->d_sizes, h->d_sw_c + b,
                                          &sb->plan_n, h->d_sw_s + b, h->d_Fall));
                HIPCHK(launch_plan_walk_many(st, p, h->d_table, h->d_sizes, h->d_state, sb, h->d_Fall, 0,
                                             h->d_sw_plans + b, 1));
            }
        }
        h->any_solve = true;
        h->timed = recorded ? alpa_dp::RECORDED : alpa_dp::TIMED;
        return ALPA_DP_OK;
    }
    HIPCHK(launch_epilogue(st, p, h->d_cand, h->d_Fmin, h->d_Sbest, h->d_state, prune_sel, d_out_T != nullptr,
                           have_list || !d_out_T ? h->d_T : d_out_T, kept, h->d_plan_tmp, h->d_best_plan, d_out_plan));
    if (d_out_T && have_list && bound > 0) HIPCHK(launch_scatter_T(st, h->d_T, h->d_rank, n_tmax, d_out_T));
    // every layer of the winning candidate (does nothing if there is none), then the walk
    if (band) {
        FastArgs fa{p_band, nullptr, h->band_shapes.sizes, &h->d_state->best_c, nullptr,
                    &h->d_state->plan_n, 0, INT32_MAX, &h->d_state->plan_ticket, &h->d_state->wave_relax,
                    nullptr, 0, 0, h->d_tmpFS, h->d_tmpFS + 2, 1, h->d_Fall, &h->d_state->best_s,
                    nullptr, bounds};
        HIPCHK(launch_recurrence_band(st, fa, h->band, h->d_bandrecs, h->d_bandends, h->d_bandthr, h->max_finite, FAST_MODE_PLAN, 1));
    } else if (h->fast_ok && p.D <= 64 && !(flags & ALPA_DP_GENERIC)) {
        FastArgs fa{p, h->d_recs, h->d_sizes, &h->d_state->best_c, nullptr,
                    &h->d_state->plan_n, 0, INT32_MAX, &h->d_state->plan_ticket, &h->d_state->wave_relax,
                    nullptr, 0, 0, h->d_tmpFS, h->d_tmpFS + 2, 1, h->d_Fall, &h->d_state->best_s,
                    h->d_gmin, nullptr};
        HIPCHK(launch_recurrence_fast(st, fa, FAST_MODE_PLAN, 1, 1));
    } else {
        HIPCHK(launch_plan_layers(st, p, h->d_table, h->d_sizes, &h->d_state->best_c,
                                  &h->d_state->plan_n, &h->d_state->best_s, h->d_Fall));
    }
    HIPCHK(launch_plan_walk(st, p, h->d_table, h->d_sizes, h->d_state, h->d_Fall, h->d_plan_tmp,
                            h->d_best_plan, d_out_plan));
    h->any_solve = true;
    h->have_best = true;
    h->timed = recorded ? alpa_dp::RECORDED : alpa_dp::TIMED;
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_solve_dev(alpa_dp_t *h, const int32_t *d_tmax, int n_tmax, unsigned flags,
                                 int64_t *d_out_T, alpa_plan_t *d_out_plan)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    return solve_dev_impl(h, d_tmax, n_tmax, flags, d_out_T, d_out_plan, 31);
}

// Checks a host candidate list and queues its copy to the device; *d_tmax stays null if
// there is none.
static int stage_host_candidates(alpa_dp *h, const int32_t *tmax, int n_tmax,
                                 const int32_t **d_tmax, int *key_bits)
{
    *d_tmax = nullptr;
    *key_bits = 31;
    if (tmax) {
        if (n_tmax == 0) return fail(ALPA_DP_EINVAL, "empty candidate list");
        int32_t mx = 0;
        for (int j = 0; j < n_tmax; ++j) {
            if (tmax[j] < 0 || tmax[j] == ALPA_DP_INF_I32)
                return fail(ALPA_DP_EINVAL, "candidate out of range");
            mx = std::max(mx, tmax[j]);
        }
        *key_bits = bits_for((uint32_t)mx);
        {
            const int rc = ensure_candidate_arrays(h, n_tmax);
            if (rc) return rc;
        }
        HIPCHK(hipMemcpyAsync(h->d_tmax_stage, tmax, (size_t)n_tmax * 4, hipMemcpyHostToDevice,
                              h->stream));
        *d_tmax = h->d_tmax_stage;
    }
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_solve(alpa_dp_t *h, const int32_t *tmax, int n_tmax, unsigned flags,
                             int64_t *out_T, alpa_plan_t *out_plan)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    if (n_tmax < 0) return fail(ALPA_DP_EINVAL, "n_tmax < 0");
    int key_bits = 31;
    const int32_t *d_tmax = nullptr;
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    {
        int rc = stage_host_candidates(h, tmax, n_tmax, &d_tmax, &key_bits);
        if (rc) return rc;
    }
    const int n_out = candidate_bound(h, tmax != nullptr, n_tmax);
    int rc = solve_dev_impl(h, d_tmax, n_tmax, flags, out_T ? h->d_outT_stage : nullptr,
                            out_plan ? h->d_plan_tmp : nullptr, key_bits);
    if (rc) return rc;
    if (out_T && n_out > 0)
        HIPCHK(hipMemcpyAsync(out_T, h->d_outT_stage, (size_t)n_out * 8, hipMemcpyDeviceToHost,
                              h->stream));
    if (out_plan)
        HIPCHK(hipMemcpyAsync(out_plan, h->d_plan_tmp, sizeof(alpa_plan_t), hipMemcpyDeviceToHost,
                              h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    if (out_plan && out_plan->num_stages < 0)
        return fail(ALPA_DP_EHIP, "internal inconsistency during plan recovery");
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_solve_sweep(alpa_dp_t *h, const int32_t *tmax, int n_tmax, unsigned flags,
                                   const int32_t *B_values, int n_B, alpa_plan_t *out_plans)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    if (n_tmax < 0) return fail(ALPA_DP_EINVAL, "n_tmax < 0");
    if (!B_values || !out_plans) return fail(ALPA_DP_EINVAL, "B_values or out_plans is null");
    if (n_B < 1 || n_B > ALPA_DP_MAX_SWEEP) return fail(ALPA_DP_EINVAL, "n_B out of range");
    for (int b = 0; b < n_B; ++b)
        if (B_values[b] < 1) return fail(ALPA_DP_EINVAL, "B must be >= 1");
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    int key_bits = 31;
    const int32_t *d_tmax = nullptr;
    int rc = stage_host_candidates(h, tmax, n_tmax, &d_tmax, &key_bits);
    if (rc) return rc;
    if (n_B > h->sw_cap) {
        HIPCHK(hipStreamSynchronize(h->stream));
        rc = alloc_sweep_arrays(h, n_B);
        if (rc) return rc;
    }
    int32_t head[2 * ALPA_DP_MAX_SWEEP];           // of every chunk: B values, ticket
    int n_head = 0;
    for (int b = 0, chunk = sweep_chunk(h, n_B); b < n_B; b += chunk) {
        head[n_head++] = std::min(chunk, n_B - b);
        head[n_head++] = 0;
    }
    HIPCHK(hipMemcpyAsync(h->d_sw_n, head, (size_t)n_head * 4, hipMemcpyHostToDevice, h->stream));
    HIPCHK(hipMemcpyAsync(h->d_sw_B, B_values, (size_t)n_B * 4, hipMemcpyHostToDevice, h->stream));
    rc = solve_dev_impl(h, d_tmax, n_tmax, flags, nullptr, nullptr, key_bits, n_B);
    if (rc) {
        (void)hipStreamSynchronize(h->stream);     // `head` above is read by a queued copy
        return rc;
    }
    HIPCHK(hipMemcpyAsync(out_plans, h->d_sw_plans, (size_t)n_B * sizeof(alpa_plan_t),
                          hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    for (int b = 0; b < n_B; ++b)
        if (out_plans[b].num_stages < 0)
            return fail(ALPA_DP_EHIP, "internal inconsistency during plan recovery");
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_candidates(alpa_dp_t *h, int32_t *out, int cap, int *out_n)
{
    if (!h || !out_n || (cap > 0 && !out)) return fail(ALPA_DP_EINVAL, "null argument");
    if (!h->any_solve) return fail(ALPA_DP_EINVAL, "no solve has been made on this handle");
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    SolveState s;
    HIPCHK(hipMemcpyAsync(&s, h->d_state, sizeof(s), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    *out_n = s.n_cand;
    const int n = std::min(cap, s.n_cand);
    if (n > 0) {
        HIPCHK(hipMemcpyAsync(out, h->d_cand, (size_t)n * 4, hipMemcpyDeviceToHost, h->stream));
        HIPCHK(hipStreamSynchronize(h->stream));
    }
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_best(alpa_dp_t *h, alpa_plan_t *out_plan)
{
    if (!h || !out_plan) return fail(ALPA_DP_EINVAL, "null argument");
    if (!h->have_best) {
        int rc = alpa_dp_solve(h, nullptr, 0, ALPA_DP_PRUNE, nullptr, nullptr);
        if (rc) return rc;
    }
    int prev = 0;
    HIPCHK(hipGetDevice(&prev));
    if (prev != h->device) HIPCHK(hipSetDevice(h->device));
    struct Restore { int prev, cur; ~Restore() { if (prev != cur) (void)hipSetDevice(prev); } }
        restore{prev, h->device};
    HIPCHK(hipMemcpyAsync(out_plan, h->d_best_plan, sizeof(alpa_plan_t), hipMemcpyDeviceToHost,
                          h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_last_timing(alpa_dp_t *h, float *ms_candidates, float *ms_recurrence,
                                   float *ms_epilogue)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    if (h->timed == alpa_dp::NOT_TIMED) return fail(ALPA_DP_EINVAL, "no solve has been made on this handle");
    if (h->timed == alpa_dp::RECORDED) return fail(ALPA_DP_EHIP, "the last solve was recorded into a graph");
    SolveState s;
    HIPCHK(hipMemcpyAsync(&s, h->d_state, sizeof(s), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    auto ms = [&](int x) { return (float)((double)(s.clock[x + 1] - s.clock[x]) / h->clock_khz); };
    if (ms_candidates) *ms_candidates = ms(0);
    if (ms_recurrence) *ms_recurrence = ms(1);
    if (ms_epilogue) *ms_epilogue = ms(2);
    return ALPA_DP_OK;
}

// For the tests that name a route (not in the public header): the graph of each interval of thresholds, eight int32 each as GraphHead has
// them, and how the candidates of the last solve with ALPA_DP_COUNT_WORK were settled (SparseRoute).  EINVAL where there are no graphs.
extern "C" int alpa_dp_routes_(alpa_dp_t *h, int32_t *heads, int32_t *routes)
{
    static_assert(sizeof(GraphHead) == 32, "eight int32");
    if (!h || !heads || !routes) return fail(ALPA_DP_EINVAL, "null argument");
    if (!h->sparse_ok || !h->have_bounds) return fail(ALPA_DP_EINVAL, "no graphs on this handle");
    SolveState s;
    HIPCHK(hipMemcpyAsync(heads, graph_heads(h->d_graph, h->p.K, h->p.D), BAND_THRESHOLDS * sizeof(GraphHead), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipMemcpyAsync(&s, h->d_state, sizeof(s), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    std::copy(s.routes, s.routes + 5, routes);
    return ALPA_DP_OK;
}

extern "C" int alpa_dp_last_counters(alpa_dp_t *h, int *n_candidates, int64_t *wave_relaxations)
{
    if (!h) return fail(ALPA_DP_EINVAL, "handle is null");
    if (!h->any_solve) return fail(ALPA_DP_EINVAL, "no solve has been made on this handle");
    SolveState s;
    HIPCHK(hipMemcpyAsync(&s, h->d_state, sizeof(s), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    if (n_candidates) *n_candidates = s.n_cand;
    if (wave_relaxations) *wave_relaxations = (int64_t)s.wave_relax;
    return ALPA_DP_OK;
}
