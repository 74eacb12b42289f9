// Internal declarations shared by the translation units of libalpa_dp (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>

namespace alpa {

// Device-side +infinity.  Finite sums stay below it (checked at create: K * max finite
// latency < 2^30) and INF + INF = 2^31 - 2 still fits in int32, so "never add to
// infinity" becomes "add, then anything >= DEV_INF is infinity".
constexpr int32_t DEV_INF = (1 << 30) - 1;
constexpr int64_t INF_I64 = INT64_MAX;
constexpr int32_t INF_I32 = INT32_MAX;

// What Fmin holds besides sums and DEV_INF (no plan): not there yet; not evaluated, as the early exit comes before; not
// evaluated, as a lower candidate has no higher T.
constexpr int32_t F_NOT_YET = -1, F_SKIPPED = DEV_INF + 1, F_LEFT_OUT = DEV_INF + 2;

constexpr int WAVE = 64;
constexpr int PRUNE_CHUNK = 64;          // candidates per published running-minimum slot

// Result block of one solve, in device memory.
struct SolveState {
    int32_t n_cand;          // distinct candidates of this solve
    int32_t ticket;          // next candidate index to hand out (recurrence kernel)
    int32_t n_processed;     // prefix length after the exact pruning rule
    int32_t best_idx;        // index of the winning candidate, -1 if none
    int64_t best_T;          // its T*
    int32_t best_c;          // its t_max
    int32_t best_s;          // its number of stages
    unsigned long long wave_relax;   // executed 64-lane relaxations (instrumented runs)
    int32_t n_distinct;      // distinct finite table values seen by candidate preparation
    int32_t plan_n;          // 1 if a plan is to be recovered (a feasible winner exists)
    int32_t plan_ticket;     // ticket counter of the plan-recovery run
    int32_t n_first;         // candidates [n_first, n_range) are searched (kernels_refine.hip)
    int32_t n_range;
    int32_t n_list;          // candidates to evaluate in the present round
    int32_t n_knots;         // candidates evaluated so far
    int32_t n_todo;          // of the present round, those that the graphs do not settle
    int32_t todo_ticket;
    int32_t thin[4];         // see recurrence_band_kernel
    int32_t n_slots;         // plans kept for the selection (kernels_sparse.hip)
    int32_t plan_done;       // the selection has written the plan
    int32_t routes[5];       // instrumented runs: see SparseRoute
    int64_t clock[4];        // the device's clock before the candidates, behind them, before the selection and at the end
};

struct Problem {
    int K, N, M, D, S, Smax, B;
};

// ---- wave-level reductions (DPP inside rows of 16, ds_swizzle across 16, bpermute across 32)

template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

// xor-16 inside each half of the wave: ds_swizzle bit mode (and 0x1f, or 0, xor 0x10)
__device__ __forceinline__ int swz_xor16(int v)
{
    return __builtin_amdgcn_ds_swizzle(v, 0x401F);
}

__device__ __forceinline__ int xor32(int v)
{
    return __shfl_xor(v, 32, 64);
}

// min over the 64 lanes, result in every lane
__device__ __forceinline__ int wave_min_i32(int v)
{
    v = min(v, dpp_mov<0xB1>(v));    // quad_perm [1,0,3,2]
    v = min(v, dpp_mov<0x4E>(v));    // quad_perm [2,3,0,1]
    v = min(v, dpp_mov<0x141>(v));   // row_half_mirror
    v = min(v, dpp_mov<0x140>(v));   // row_mirror
    v = min(v, swz_xor16(v));
    v = min(v, xor32(v));
    return v;
}

__device__ __forceinline__ int64_t i64_from(int lo, int hi)
{
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ int lo32(int64_t v) { return (int)(uint32_t)(uint64_t)v; }
__device__ __forceinline__ int hi32(int64_t v) { return (int)((uint64_t)v >> 32); }

template <int CTRL>
__device__ __forceinline__ int64_t dpp_mov64(int64_t v)
{
    return i64_from(dpp_mov<CTRL>(lo32(v)), dpp_mov<CTRL>(hi32(v)));
}

__device__ __forceinline__ int64_t min64(int64_t a, int64_t b) { return a < b ? a : b; }

__device__ __forceinline__ int64_t wave_min_i64(int64_t v)
{
    v = min64(v, dpp_mov64<0xB1>(v));
    v = min64(v, dpp_mov64<0x4E>(v));
    v = min64(v, dpp_mov64<0x141>(v));
    v = min64(v, dpp_mov64<0x140>(v));
    v = min64(v, i64_from(swz_xor16(lo32(v)), swz_xor16(hi32(v))));
    v = min64(v, i64_from(xor32(lo32(v)), xor32(hi32(v))));
    return v;
}

// inclusive prefix minimum over the 64 lanes (lane l gets min of lanes 0..l)
__device__ __forceinline__ int64_t wave_prefix_min_i64(int64_t v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int lo = __shfl_up(lo32(v), off, 64);
        const int hi = __shfl_up(hi32(v), off, 64);
        const int64_t o = i64_from(lo, hi);
        if (lane >= off) v = min64(v, o);
    }
    return v;
}

// Next ticket of a work counter, drawn by one thread of the workgroup (`tid` == 0) and handed to all of
// them through *sh.  Two barriers.  The thread id goes through an opaque register on every call: a
// branch on it inside a persistent loop is otherwise loop-invariant, the compiler splits the loop on
// it, and the lanes of one wave then run the loop out of step with each other.  (All threads adding 0 but
// one needs no branch, but is 64 serial operations a wave on one address: 512 workgroups of sixteen
// waves spent 65 us there before their first candidate.)
__device__ __forceinline__ int draw_ticket(int32_t *ticket, int tid, int32_t *sh)
{
    int t = tid;
    asm volatile("" : "+v"(t));
    if (t == 0) *sh = atomicAdd(ticket, 1);
    __syncthreads();
    const int tk = __builtin_amdgcn_readfirstlane(*sh);
    __syncthreads();
    return tk;
}

// atomicMin by one thread of the workgroup (see draw_ticket)
__device__ __forceinline__ void publish_min(int64_t *p, int64_t v, int tid)
{
    int t = tid;
    asm volatile("" : "+v"(t));
    if (t == 0) atomicMin((long long *)p, (long long)v);
}

// Barrier for what the waves exchange through LDS: loads from global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- host-side launchers (callers validate sizes first; none of these synchronises)

constexpr int SORT_SLICES = 1024;        // one-wave slices of the radix sort
constexpr int SORT_RADIX = 256;          // 8-bit digits

struct PrepBuffers {
    int32_t *keys[2];        // [capacity] each
    uint32_t *hist;          // [SORT_RADIX * SORT_SLICES] slice counts + [SORT_RADIX] digit totals
    uint32_t *block_cnt;     // [capacity / 4096 + 2]
};

hipError_t launch_gather_table_values(hipStream_t st, const int32_t *table, int K, int S,
                                      int32_t inf_key, int32_t *out_keys);
hipError_t launch_sort_dedup(hipStream_t st, PrepBuffers &pb, int n, int key_bits,
                             int32_t drop_key, int32_t *out_unique, uint32_t *out_n_unique);
// Values up to these go through a presence bitmap instead of the sort: one in LDS (64 KiB), merged into the global
// one, or the global one alone.
constexpr int32_t DISTINCT_LOCAL_MAX = 1 << 19, DISTINCT_BITMAP_MAX = 1 << 25;
hipError_t launch_bitmap_clear(hipStream_t st, uint32_t *work, int32_t max_value);
// lists up to this long are sorted by one block
constexpr int LIST_SORT_MAX = 8192;
hipError_t launch_list_sort(hipStream_t st, const int32_t *tmax, int n, int32_t *out_unique, uint32_t *out_n_unique,
                            SolveState *state, int32_t *rank_of_orig);
hipError_t launch_distinct_by_bitmap(hipStream_t st, const int32_t *table, int K, int S,
                                     int32_t max_value, uint32_t *work, int32_t *out_unique,
                                     uint32_t *out_n_unique);
size_t distinct_bitmap_words(int32_t max_value);

// What is known of a table for certain values of t_max (kernels_band.hip): the thresholds, from no filter at all
// and the largest latency down, sixteen an octave.
constexpr int BAND_THRESHOLDS = 120;
__host__ __device__ __forceinline__ int32_t band_threshold(int32_t max_finite, int j)
{
    if (j == 0) return DEV_INF - 1;
    return (int32_t)(((int64_t)max_finite * (32 - ((j - 1) & 15)) >> 5) >> ((j - 1) >> 4)) + 1;
}
// behind the bounds (launch_band_bounds): a lower bound on F for each threshold and the least largest stage; then the sum and the
// largest latency of a plan for each, room for 2 BAND_THRESHOLDS + 1 more, and what is there for the present table: 1 for these
// numbers, 2 and 4 for the two halves of launch_band_exact_bounds; and whether latencies fall with the number of stages
constexpr int BAND_THERE = 5 * BAND_THRESHOLDS + 2, BAND_FALLS = BAND_THERE + 1, BAND_TOTALS = BAND_FALLS + 1;

// Rounds of evaluation (kernels_refine.hip)
constexpr int REFINE_MAX_KNOTS = 4096;   // knots a refinement step takes in (LDS)
struct RefineBuffers {
    int32_t *knots[2];       // [REFINE_MAX_KNOTS] each: positions evaluated so far, ascending
    int32_t *list;           // [candidate capacity] positions to evaluate in the present round
    int all;                 // up to so many candidates worth searching: one round takes them all
    int first_round;         // else: knots of the first round
    int budget;              // points of a round that is neither the first nor the last
    int rounds;              // launched; those behind one that has settled everything are empty
};
// What is asked of the candidates: per-candidate results, or the plan alone for one or several B values
struct RefineQuery {
    const int32_t *B_vals;   // device array of n_B values, or null: B
    int B, n_B;
    int prune;               // the early exit of Alg. 1 (one B value)
    int plan_only;
    const int32_t *bounds;   // launch_table_bounds
    int Smax;
    int early_exit;          // the selection uses the early exit (in a sweep too, where `prune` is not set)
    const int32_t *thr;      // BAND_TOTALS numbers of launch_band_bounds, or null
    int32_t max_finite;
    const struct GraphHead *heads;   // of the table's graphs, where fewer knots do if many candidates have none (or null)
};
// `bound`: the host's upper bound of the number of candidates
// candidates from the table's distinct values (distinct null: they are there)
struct PickQuery {
    const int32_t *distinct;
    const uint32_t *n_distinct;
    int n_quantiles, cap;
};
hipError_t launch_pick_candidates(hipStream_t st, PickQuery &pick, int bound, int32_t *cand, SolveState *state);
hipError_t launch_set_candidates(hipStream_t st, const uint32_t *n_unique, SolveState *state);
// first round: the range worth searching and its knots
hipError_t launch_refine_begin(hipStream_t st, const RefineQuery &rq, const PickQuery &pick, int32_t *cand, SolveState *state,
                               const RefineBuffers &rb);
// the step behind round `round` (1-based)
hipError_t launch_refine(hipStream_t st, const RefineQuery &rq, const int32_t *cand, int32_t *Fmin,
                         SolveState *state, int round, int last, const RefineBuffers &rb);
hipError_t launch_rank_lookup(hipStream_t st, const int32_t *tmax, int n, const int32_t *unique,
                              const uint32_t *n_unique, int32_t *rank_of_orig);

// table[s-1][k][i][q] from profiled options [k][i][q][o]; *max_finite = largest finite entry
// (-1 if none).  O * 1 KiB of LDS per block: O <= 32.
hipError_t launch_build_table(hipStream_t st, const int32_t *t_l, const int64_t *mem_stage,
                              const int64_t *mem_act, int K, int S, int O, int64_t mem_device,
                              int32_t *table, int32_t *max_finite);

// out[0] = smallest, out[1] = largest finite entry (-1 if none) of the used part of a table, out[2] = 1 if one is below that of fewer
// stages (of up to Smax)
hipError_t launch_table_range(hipStream_t st, const int32_t *table, int K, int S, int Smax, int32_t *out);

hipError_t launch_valu_peak(hipStream_t st, int grid, int iters, int32_t *sink);
hipError_t launch_equal_layer_mask(hipStream_t st, int32_t *table, int K, int S);

hipError_t launch_repack_fast(hipStream_t st, const int32_t *table, int K, int D, int S, int KP,
                              int32_t *recs, int32_t *group_min);
size_t fast_table_ints(int K, int S);    // size of the column-record array, padding included
int fast_group_min_stages(int K, int D);        // stage counts the early-stop table spans
size_t fast_group_min_ints(int K, int D, int S);   // size of the early-stop table

hipError_t launch_recurrence_generic(hipStream_t st, const Problem &p, const int32_t *table,
                                     const int32_t *sizes, const int32_t *cand, const int32_t *list,
                                     const int32_t *n_list_p, int32_t *ticket, int64_t *chunk_min,
                                     int prune, int32_t *Fmin, int32_t *Sbest, int32_t *scratch,
                                     int n_layers, const int32_t *s_bound, int grid);
struct FastArgs {
    Problem p;
    const int32_t *recs, *sizes, *cand;
    // positions in `cand` to evaluate, ascending, and their number (device memory); the plan mode
    // takes candidates 0 .. *n_list_p - 1 instead.  The launch does nothing unless
    // n_lo < *n_list_p <= n_hi.
    const int32_t *list, *n_list_p;
    int n_lo, n_hi;
    int32_t *ticket;
    unsigned long long *wave_relax;
    int64_t *chunk_min;
    int prune, descending;
    int32_t *Fmin, *Sbest;
    int dummy_idx;           // spare slot of Fmin / Sbest for the waves that own no result
    // plan mode only: candidate j dumps its layers to F_all + j * (Smax+1) * (K+2)*(D+1) and
    // stops at layer s_top_p[j], the winner's number of stages (device memory)
    int32_t *F_all;
    const int32_t *s_top_p;
    const int32_t *group_min;   // early-stop table (launch_repack_fast)
    const int32_t *s_bound;     // [Smax + 1]: the least unfiltered F of more than s stages (batch modes)
    // batch modes, one-candidate form: 0, or the width DP of the lane groups
    // (a power of two, D <= DP <= 32): 64 / DP candidates per workgroup
    int grouped = 0;
    // band kernel: the list that `list` is what is left of, ascending (null: none), and, where a candidate that a lower one beats for
    // every B value need not be evaluated, those values (n_B of them, or null: p.B)
    const int32_t *whole = nullptr, *n_whole_p = nullptr;
    int32_t *rest = nullptr, *thin = nullptr;      // room for as many as `list` has; SolveState::thin
    bool leave_out = false;
    const int32_t *B_vals = nullptr;
    int n_B = 0;
};
// narrowest lane group that holds a mesh of D devices
inline int fast_lane_group_width(int D)
{
    int dp = 1;
    while (dp < D) dp <<= 1;
    return dp;
}
// more than 64 devices: from this many waves along the first layers on (81 layers)
constexpr int FAST_WIDE_NWK = 6;
enum { FAST_MODE_BATCH = 0, FAST_MODE_COUNT = 1, FAST_MODE_PLAN = 2, FAST_MODE_FEW = 3 };
hipError_t launch_recurrence_fast(hipStream_t st, const FastArgs &a, int mode, int nc, int grid);
int fast_kernel_blocks_per_cu(int K, int nc);
// the instances for 65-128 layers (kernels_fast_deep.hip)
hipError_t launch_recurrence_fast_deep(hipStream_t st, const FastArgs &a, int mode, int nc, int grid);
int fast_kernel_blocks_per_cu_deep(int K, int nc);

// a workgroup per candidate, t_intra in bands by row broadcast (kernels_band.hip)
constexpr int BAND_THIN_FROM = 512;            // more left than that: knots first, from the whole list (up to two a compute unit run at once)
struct BandShape {
    int nbuf;                // F buffers in LDS; 0: the problem does not fit
    int W;                   // windows of 64 device counts
    int ahead, cap;          // layers whose work lists are made at a time; units a layer can have
    int lens_at, bounds_at, lds_ints;   // in int32: where a candidate's stage lengths and its windows are kept; all of the LDS
};
BandShape band_shape(int K, int D, int S, const int32_t *sizes);
// The shapes as the band kernel sees them: one per device count.  Shapes first[q], next[first[q]], .. of the table up to -1
// have sizes[q] devices; first is null where the table has no two of a kind.
struct BandShapes {
    int S, S_table;
    const int32_t *sizes, *first, *next;
};
// The smallest of an entry's shapes of one device count: `entry` is that of shape 0.  What a filter leaves of several shapes
// with equal device counts has the least sum with the smallest of them, so the kernel sees one shape for each.
__device__ __forceinline__ int32_t band_smallest(const int32_t *__restrict__ entry, const BandShapes &b, int q)
{
    if (!b.first) return entry[q];
    int32_t t = INF_I32;
    for (int x = b.first[q]; x >= 0; x = b.next[x]) t = min(t, entry[x]);
    return t;
}

size_t band_table_ints(int K, int Smax, int S);
size_t band_ends_ints(int K, int Smax, int S);
hipError_t launch_repack_band(hipStream_t st, const int32_t *table, const Problem &p, const BandShapes &b,
                              int32_t *recs, int32_t *ends, int32_t *bounds, bool falls);
// what the table says about candidates: launch_table_bounds' place for these sizes; `once`: nothing is done where it is there
// (a recorded solve is replayed)
size_t band_thresholds_ints(int K, int D);
struct BandWork {
    const int32_t *least, *front;  // front_least_ints, front_table_ints, of launch_front_table
    int32_t *thr, *backs;    // band_thresholds_ints each (no windows in the second)
    int32_t *graph;          // graph_table_ints; null where candidates do not go by graphs
};
hipError_t launch_band_bounds(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                              const BandWork &w, int32_t *bounds, bool once);
hipError_t launch_band_exact_bounds(hipStream_t st, const BandShapes &b, const BandShape &shape, const Problem &p, int32_t max_finite,
                                    const int32_t *recs, const int32_t *ends, int32_t *work, const int32_t *thr, int32_t *bounds, bool once);
hipError_t launch_recurrence_band(hipStream_t st, const FastArgs &f, const BandShape &b, const int32_t *recs,
                                  const int32_t *ends, const int32_t *thr, int32_t max_finite, int mode, int grid);

// front costs (kernels_front.hip)
struct FrontTable {
    const int32_t *units, *unit_min, *least;
    const uint8_t *run;
    const int32_t *sizes;
    int NG;
};
size_t front_least_ints(int K, int S);
size_t front_table_ints(int K, int S);
size_t front_lds_bytes(int K, int D, int S);
FrontTable front_table(const int32_t *least, const int32_t *front, int K, int S, const int32_t *sizes, bool back);
hipError_t launch_front_table(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t *work, int32_t *front);
hipError_t launch_front_thresholds(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                                   const int32_t *work, const int32_t *front, int32_t *fronts, int32_t *backs, int32_t *totals,
                                   int32_t *plans, int32_t *windows, int32_t *graph_used, const int32_t *asked);

// candidates by the stages that can be in their best plans (kernels_sparse.hip)
struct GraphHead { int first, n_stages, n_cells, n_chunks, from, twice, pad[2]; };      // see kernels_sparse.hip; n_stages < 0: no graph
const GraphHead *graph_heads(int32_t *graph, int K, int D);
constexpr int SPARSE_PLANS = 4096;       // plans that are kept for the selection, K uint16 each
// how sparse_eval_kernel has settled a candidate
enum SparseRoute { ROUTE_BELOW, ROUTE_PASS, ROUTE_SECOND_PASS, ROUTE_LAYERS, ROUTE_LEFT };
struct SparseOut {
    int32_t *todo, *n_todo;  // candidates that are left to the recurrence
    int32_t *slot, *n_slots; // each candidate's plan (-1: not kept)
    uint16_t *plans;         // its stages in the graph that it is from
    int32_t *plan_from;      // where that begins
    int32_t *routes;
};
size_t graph_table_ints(int K, int D);
int32_t *graph_used(int32_t *graph, int K, int D);
const int4 *graph_stages(int32_t *graph, int K, int D);
hipError_t launch_sparse_graph(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                               const int32_t *work, const int32_t *front, const int32_t *fronts, const int32_t *backs,
                               const int32_t *totals, int32_t *plans, const int32_t *falls, int32_t *graph, int32_t *bounds, int32_t *there, bool once);
// f: the recurrence's arguments (those of them that count); most: upper bound of the list's length
hipError_t launch_sparse_eval(hipStream_t st, const FastArgs &f, const int32_t *table, int32_t *graph, int32_t max_finite, const SparseOut &o, bool count,
                              int most, int n_cu);

// plan recovery of one candidate, a launch per layer (general sizes)
hipError_t launch_plan_layers(hipStream_t st, const Problem &p, const int32_t *table,
                              const int32_t *sizes, const int32_t *c_p, const int32_t *n_p,
                              const int32_t *s_top_p, int32_t *F_all);
// bounds of the table (kernels_generic.hip): [0..Smax] the least unfiltered F of more than s stages, then
// the smallest t_max with a plan and the stages of one; work: table_bounds_work() int32
inline size_t table_bounds_ints(const Problem &p) { return (size_t)p.Smax + 4; }
inline size_t table_bounds_work(const Problem &p)
{
    return 4 * (size_t)(p.K + 2) * (p.D + 1) + 2 * ((size_t)p.Smax + 1);
}
hipError_t launch_table_bounds(hipStream_t st, const Problem &p, const int32_t *table,
                               const int32_t *sizes, int32_t *work, int32_t *bounds);
// plans of the candidates that the graphs have settled (slot null: of none)
struct KeptPlans {
    const int32_t *slot;
    const uint16_t *plans;
    const int32_t *from;
    const int4 *stages;      // of all graphs (kernels_sparse.hip)
};
hipError_t launch_epilogue(hipStream_t st, const Problem &p, const int32_t *cand,
                           const int32_t *Fmin, const int32_t *Sbest, SolveState *state, int prune,
                           bool want_T, int64_t *T, const KeptPlans &kept, void *plan_tmp, void *best_plan, void *plan_out);
hipError_t launch_scatter_T(hipStream_t st, const int64_t *T, const int32_t *rank_of_orig,
                            int n_orig, int64_t *out_T);
hipError_t launch_plan_walk(hipStream_t st, const Problem &p, const int32_t *table,
                            const int32_t *sizes, SolveState *state, const int32_t *F_all,
                            void *plan_tmp, void *best_plan, void *plan_out);
// sweep over B: one block per B value
hipError_t launch_sweep_epilogue(hipStream_t st, const int32_t *B_vals, int n_B,
                                 SolveState *solve, const int32_t *cand,
                                 const int32_t *Fmin, const int32_t *Sbest, SolveState *states,
                                 int prune, int32_t *win_c, int32_t *win_s, const Problem &p, const KeptPlans &kept, void *plans);
hipError_t launch_plan_walk_many(hipStream_t st, const Problem &p, const int32_t *table,
                                 const int32_t *sizes, SolveState *solve, SolveState *states, const int32_t *F_all,
                                 size_t slab, void *plans, int n);
hipError_t launch_init_state(hipStream_t st, SolveState *state, int64_t *chunk_min, int n_chunks, uint32_t *clear, int words);
hipError_t launch_init_best_plan(hipStream_t st, void *best_plan);

// operator clustering (Eq. 6).  Work memory, see kernels_cluster.hip: band [width][K], rows G and V of one
// launch, pf and win [K + 1], tot [K], arg [L][K + 1].
struct ClusterWork {
    int64_t *band, *G, *V, *pf, *tot, *keep;
    int32_t *win, *arg, *meta;
};
size_t cluster_work_i64(int K, int L, int width);
ClusterWork cluster_work(int64_t *base, int K, int L, int width);
int cluster_band_width(const int32_t *flop, int K, int64_t cap);
// width: at least the largest number of feasible first operators (K if unknown).  ctl == nullptr: the
// caller has checked the inputs and passes the FLOP bound `cap`.  ctl != nullptr ([2] int64):
// the inputs are checked and the bound is computed from delta_ppm on the device, and `cap` is
// ignored.  out is [3]: G, V, status.  exact != 0 (host-checked inputs only): a second run of
// the recurrence minimises V over every clustering that reaches G(K, L).  max_spins: how often a wait
// between workgroups looks for its value before it gives up (about 0.5 us a look; waits take a few, unless
// another call writes the same work memory).
constexpr unsigned CLUSTER_MAX_SPINS = 1u << 23;
hipError_t launch_cluster(hipStream_t st, const int32_t *flop, const int32_t *src,
                          const int32_t *dst, const int64_t *nbytes, int E, int K, int L,
                          int64_t cap, int width, const ClusterWork &w, int64_t *out,
                          int32_t *first_op, int64_t *ctl = nullptr, int delta_ppm = 0, int exact = 0,
                          unsigned max_spins = CLUSTER_MAX_SPINS);

}  // namespace alpa
