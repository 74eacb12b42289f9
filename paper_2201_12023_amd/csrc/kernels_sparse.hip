// Candidates by the few stages that can be in their best plans.
//
// Between two neighbouring thresholds of t_max (kernels_front.hip) the upper one bounds every plan from below: one that goes
// through the stage of layers k .. i on a devices with d behind its beginning is not below
//     P(k, D - d) + least(k, i, a) + Q(i + 1, d - a),
// and a plan whose stages pass the lower threshold bounds the best one from above, by U.  What is not above U is a
// graph of some ten to some thousand stages between as many cells (k, d) (64 layers on 8 x 8 of an expert model: 10 to 5100 of
// 23 000 stages on up to 64 device counts each), and every best plan of every candidate between the two is a way through
// it.  So a candidate is one pass over the graph from the last layer to the first by one wave, with its filter:
// for each cell the least sum, the fewest stages that reach it, and of those the first stage in Eq. 3's order.
//
// Latencies must not fall with the number of stages behind (checked when the handle is made; of tables built from profiled options
// they never do).  Then `run` says up to how many a stage has its least latency.  The pass takes only stages as they are (s <=
// run), so what it finds is a plan; if it had to leave one out, a second pass that leaves none out says whether that plan is
// the best all the same.  If it is not, Eq. 3 itself runs on the graph, a layer for each number of stages.  At the low end, where
// no plan is known at the lower threshold, the graph is of all stages on plans under the upper one's filter.  If a graph is too
// large its candidates go to the recurrence (kernels_band.hip).
//
// On ties: of the plans with the least sum, min_s F of Eq. 3 takes the fewest stages, and the walk from the first stage on
// the lowest last layer, then the lowest shape.  A cell on such a plan has the fewest stages of all ways of its sum (else the plan
// would have fewer), so the order of (sum, stages, last layer, shape) in each cell's own minimum is that of the walk.
#include "bounds.hpp"
#include "front.hpp"
#include "graph_label.hpp"

namespace alpa {

// Limits (first call on a table and later ones, us):
// * GRAPH_CELLS (graph_label.hpp): 96 layers on 8 x 8, all values 541 and 215, with 1024 cells 709 and 365; with 2048, and two
//   workgroups of labels to a compute unit instead of three, 560 and 220.
// * GRAPH_STAGES: a pass over so many is some 300 chunks of 0.25 us, about what the recurrence takes of a candidate.
// * GRAPH_SEARCH: 25 layers on 12 x 16, the plan out of 440 candidates 321 and 114, with 1024 and with 512 350 and 170, where those below the
//   least t_max with a plan go to the recurrence; 64 on 8 x 8 354 and 149, with 512 347 and 156; 16384 takes first calls longer (5 of 354).
// * GRAPH_LAYERS: with 128 and with 2048 the same within 3 % on 29 calls.
constexpr int GRAPH_STAGES = 1 << 14;          // of one graph
constexpr int GRAPH_CHUNKS = 512;              // of up to 64 stages that begin with one layer (at most 248 + 16384 / 64)
constexpr int GRAPH_THREADS = WAVE * FRONT_WAVES;
constexpr int GRAPH_SEARCH = 4096;             // stages of a graph in which the least t_max with a plan is looked for
constexpr int GRAPH_LAYERS = 512;              // stages of a graph on which Eq. 3 is run
constexpr int GRAPH_LDS = 128 * 1024;          // of the workgroup that makes a graph, if its list of stages takes so much

// Room for the stages of all graphs (what does not find room goes to the recurrence; which graphs find it where it is short depends on
// the order in which workgroups get there).  Graphs lie on up to K D cells: models of 24 to 200 layers on 2 x 8 to 32 x 8 take 56 to 81 000
// stages, 48 layers on 32 x 8 74 000 (with room for 28 000, 16 candidates 329 us, now 125), 100 on 12 x 8 81 000.  More room at few layers is only
// for latencies without structure, where the recurrence is the faster way (24 layers on 2 x 8, a list of 4096 256 us, 285 with all graphs).
static int graph_room(int K, int D) { return std::min(std::max({12 * K * K, 8 * K * D, 8192}), 3 << 16); }

// graphs[j] of the candidates up to threshold j; stages by cell (falling first layer, rising devices), then rising last layer and
// shape, in chunks that begin with one layer.  A stage: least latency; byte of its cell's label | byte of that of the cell behind
// << 16; what it adds to the lower half of a label; first layer << 22 | last layer << 14 | shape << 8 | run
// GraphHead::from: candidates below that have no plan at all; twice: more stages than the list held, so its cells were looked at again
struct GraphTable {
    GraphHead *heads;
    int32_t *chunks;         // [BAND_THRESHOLDS][GRAPH_CHUNKS] where each starts, and their end
    int32_t *cells;          // [BAND_THRESHOLDS][GRAPH_CELLS] where a cell's stages start
    int4 *stages;
    int32_t *used;
    int room;
};

size_t graph_table_ints(int K, int D)
{
    return (size_t)BAND_THRESHOLDS * (8 + GRAPH_CHUNKS + GRAPH_CELLS) + 4 * (size_t)(graph_room(K, D) + WAVE) + 4;
}

static GraphTable graph_table(int32_t *base, int K, int D)
{
    GraphTable g;
    g.room = graph_room(K, D);
    g.heads = (GraphHead *)base;
    g.stages = (int4 *)(base + 8 * BAND_THRESHOLDS);
    g.chunks = (int32_t *)(g.stages + g.room + WAVE);      // (a wave reads up to 64 stages behind its own)
    g.cells = g.chunks + BAND_THRESHOLDS * GRAPH_CHUNKS;
    g.used = g.cells + BAND_THRESHOLDS * GRAPH_CELLS;
    return g;
}
int32_t *graph_used(int32_t *graph, int K, int D) { return graph_table(graph, K, D).used; }
const GraphHead *graph_heads(int32_t *graph, int K, int D) { return graph_table(graph, K, D).heads; }

// Exclusive prefix sum over the block, and the total.
__device__ __forceinline__ int graph_scan(int v, int *sh, int &total)
{
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const int o = __shfl_up(x, off, WAVE);
        if (lane >= off) x += o;
    }
    __syncthreads();                                   // sh may still be read from the last call
    if (lane == WAVE - 1) sh[w] = x;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < FRONT_WAVES; ++k) {
        const int t = sh[k];
        base += k < w ? t : 0;
        total += t;
    }
    return base + x - v;
}

// The graph of interval j.  Bound by what is looked at of each cell's stages, so that is done once, up to the last layer that the
// filter lets a stage reach, by as many neighbouring cells to a wave as to any other, with 256 latencies of their first layer at a time in
// registers for all of them (read again for each cell: 57 layers on 32 x 8 522 us, now 399); what is found is listed in LDS, and only a graph of more stages than the list holds is looked at again.  (64 layers on
// 8 x 8: every cell twice and to the last layer 156 us, listed 78, now 71; on 16 x 8 209, 86 and 75; 128 layers 308, 174 and
// 118; 48 layers on 32 x 8, with front costs of its own for the lowest interval, 520, 210 and 198.)
template <int W>
__device__ __forceinline__ void sparse_graph(int j, const FrontTable &ft, const int32_t *__restrict__ table, const BandShapes &bs, int K, int D,
                                             int32_t max_finite, const int32_t *__restrict__ fronts, const int32_t *__restrict__ backs,
                                             const int32_t *__restrict__ totals, const int32_t *plans, const int32_t *__restrict__ falls,
                                             const GraphTable &g, int list_room)
{
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];
    __shared__ int sh_scan[FRONT_WAVES], sh_first;
    __shared__ int32_t sh_U, sh_plan[2];
    __shared__ uint16_t sh_cell[GRAPH_CELLS];      // cells in order: position in a [K][RS] array
    __shared__ int sh_at[GRAPH_CELLS + 1];         // where their stages start
    __shared__ int32_t sh_room[GRAPH_CELLS];       // for a stage and what is behind it
    __shared__ int sh_size[64], sh_listed;
    __shared__ int16_t sh_reach[256];              // the last layer that a stage which begins with k reaches in the interval
    constexpr int RS = WAVE * W;
    int lane = threadIdx.x & (WAVE - 1);
    const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = bs.S, SP = front_padded(S), N = K * RS;
    const int32_t single = __builtin_amdgcn_readfirstlane(front_single(table, bs, K, D)), c = min(band_threshold(max_finite, j), single);
    const int32_t low = j + 1 < BAND_THRESHOLDS ? band_threshold(max_finite, j + 1) : 0, feasible = __builtin_amdgcn_readfirstlane(totals[BAND_THRESHOLDS]);
    auto none = [&]() {
        if (tid == 0) g.heads[j] = GraphHead{0, -1};
    };
    if (*falls || totals[j] >= DEV_INF) return none();
    if (tid == 0) {
        sh_U = single <= max(low, feasible) ? single : INT32_MAX;
        sh_plan[0] = sh_plan[1] = DEV_INF;
    }
    if (tid < S) sh_size[tid] = bs.sizes[tid];
    __syncthreads();
    if (tid < BAND_THRESHOLDS && plans[2 * tid + 1] <= max(low, feasible)) atomicMin(&sh_U, plans[2 * tid]);
    __syncthreads();
    // cells on plans up to U, by falling first layer and rising devices; the end is cell 0
    const int32_t *const P = fronts + (size_t)j * N;
    int32_t *const Q = lds;                        // [K][RS]
    uint16_t *const id = (uint16_t *)(lds + N);    // [K][RS]
    // the stages as they are found: cell << 14 | number among all of its layers and shapes, and the place among the cell's
    uint32_t *const listed = (uint32_t *)(lds + N + N / 2);
    uint16_t *const listed_at = (uint16_t *)(listed + list_room);
    const int per = (N + GRAPH_THREADS - 1) / GRAPH_THREADS;
    auto place = [&](int y) { return (K - 1 - y / RS) * RS + y % RS; };
    // (in front of the first layer there is one cell, all devices: P(0, 0) = 0)
    auto front_of = [&](int x) { return x >= RS ? P[x] : x == D - 1 ? 0 : DEV_INF; };
    const int inv = (1 << 20) / S + 1;             // x / S for x < 2^14 (S <= 64)
    int n_cells, n_stages, at;
    int32_t U = __builtin_amdgcn_readfirstlane(sh_U);
    for (int k = wid; k < K; k += FRONT_WAVES) {
        const int n = (K - k) * SP;
        const int32_t *const row = ft.least + (uint32_t)((k * K + k) * SP);
        int reach = -1;
        for (int y0 = 0; y0 < n; y0 += 4 * WAVE) {
            int32_t t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = row[min(y0 + u * WAVE + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t lanes = __ballot(t[u] <= c);
                if (lanes) reach = min(y0 + u * WAVE + 63 - __clzll((long long)lanes), n - 1);
            }
        }
        if (lane == 0) sh_reach[k] = (int16_t)(reach < 0 ? -1 : k + reach / SP);
    }
    // The stages of the wave's cells: found(cell, how many it has so far, lanes that have one, whether this one has, its number), each cell's
    // in order.  Neighbouring cells mostly begin with the same layer: up to 64 of them are gone through with 256 of its latencies in
    // registers before the next 256 are read.  counts: zeros
    auto stages = [&](int *counts, auto found) {
        const int to = 1 + (n_cells - 1) * (wid + 1) / FRONT_WAVES;
        for (int a = 1 + (n_cells - 1) * wid / FRONT_WAVES; a < to;) {
            const int k = __builtin_amdgcn_readfirstlane(sh_cell[a] / RS);
            const uint64_t others = __ballot(a + lane >= to || sh_cell[min(a + lane, to - 1)] / RS != k);
            const int b = a + (others ? __ffsll((unsigned long long)others) - 1 : WAVE), n = (sh_reach[k] + 1 - k) * S;
            const int32_t *const row = ft.least + (uint32_t)((k * K + k) * SP);
            for (int y0 = 0; y0 < n; y0 += 4 * WAVE) {
                int32_t t[4];
                int at[4];                         // last layer << 16 | devices
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int y = min(y0 + u * WAVE + lane, n - 1), l = (int)(((int64_t)y * inv) >> 20);
                    const int q = y - l * S;
                    t[u] = y0 + u * WAVE + lane < n ? row[(uint32_t)(l * SP + q)] : INF_I32;
                    at[u] = (k + l) << 16 | sh_size[q];
                }
                for (int cell = a; cell < b; ++cell) {
                    const int d = sh_cell[cell] % RS + 1, before = __builtin_amdgcn_readfirstlane(counts[cell]);
                    const int32_t room = sh_room[cell];
                    int m = before;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (y0 + u * WAVE >= n) continue;          // (uniform)
                        const int i = at[u] >> 16, left = d - (at[u] & 0xffff), behind = (i + 1) * RS + left - 1;
                        const bool end = i == K - 1;
                        bool ok = t[u] <= c && (end ? left == 0 : left > 0);
                        const int32_t f = ok && !end ? Q[behind] : 0;
                        ok = ok && f < DEV_INF && t[u] + f <= room;
                        const uint64_t lanes = __ballot(ok);
                        if (lanes == 0) continue;
                        found(cell, m, lanes, ok, y0 + u * WAVE + lane);
                        m += __popcll(lanes);
                    }
                    if (m != before && lane == 0) counts[cell] = m;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            }
            a = b;
        }
    };
    for (int turn = 0;; ++turn) {
        // (opaque: what is computed of it would be kept in registers through the front costs below)
        int me = tid;
        asm volatile("" : "+v"(me));
        lane = me & (WAVE - 1);
        for (int x = me; x < N; x += GRAPH_THREADS) {
            const int32_t p = front_of(x), q = backs[(size_t)j * N + x];
            Q[x] = p < DEV_INF && q < DEV_INF && p + q <= U ? q : DEV_INF;
        }
        if (me == 0) sh_listed = 0;
        __syncthreads();
        int mine = 0;
        for (int y = me * per; y < min(me * per + per, N); ++y) mine += Q[place(y)] < DEV_INF;
        at = 1 + graph_scan(mine, sh_scan, n_cells);
        ++n_cells;
        n_stages = GRAPH_STAGES + 1;
        if (n_cells <= GRAPH_CELLS) {              // (uniform)
            for (int y = me * per; y < min(me * per + per, N); ++y) {
                const int x = place(y);
                if (Q[x] < DEV_INF) {
                    sh_cell[at] = (uint16_t)x;
                    sh_at[at] = 0;
                    sh_room[at] = U - front_of(x);
                    id[x] = (uint16_t)at++;
                }
            }
            __syncthreads();
            // how many stages each has: as many cells for every wave
            stages(sh_at, [&](int cell, int n, uint64_t lanes, bool ok, int y) {
                int to = 0;
                if (lane == 0) to = atomicAdd(&sh_listed, __popcll(lanes));
                const int before = __popcll(lanes & ((1ull << lane) - 1)), e = __builtin_amdgcn_readfirstlane(to) + before;
                if (ok && e < list_room) {
                    listed[e] = (uint32_t)cell << 14 | (uint32_t)y;
                    listed_at[e] = (uint16_t)(n + before);
                }
            });
            __syncthreads();
            constexpr int EACH = (GRAPH_CELLS + GRAPH_THREADS - 1) / GRAPH_THREADS;
            int own[EACH], sum = 0;
#pragma unroll
            for (int u = 0; u < EACH; ++u) {
                const int x = me * EACH + u;
                own[u] = x >= 1 && x < n_cells ? sh_at[x] : 0;
                if (own[u] >= 1 << 13) own[u] = GRAPH_STAGES + 1;          // (a label has 13 bits for its number)
                sum += own[u];
            }
            at = graph_scan(sum, sh_scan, n_stages);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < EACH; ++u) {
                const int x = me * EACH + u;
                if (x < n_cells) sh_at[x] = at;
                at += own[u];
            }
            if (me == 0) sh_at[n_cells] = n_stages;               // (n_cells <= GRAPH_CELLS)
        }
        __syncthreads();
        if (n_stages <= GRAPH_STAGES) break;
        // too large: in the lowest interval a plan at the least t_max that admits any may bound it
        if (turn > 0 || low >= feasible) return none();
        const FrontLds l = front_lds(lds, K, D, ft.NG, W);
        front_costs<W, FRONT_WAVES, 0, false>(ft, K, D, S, min(feasible, single), l);
        front_plan(ft, table, bs, K, D, min(feasible, single), l.P, sh_plan);
        __syncthreads();
        if (sh_plan[1] > feasible || sh_plan[0] >= U) return none();
        U = __builtin_amdgcn_readfirstlane(sh_plan[0]);
    }
    if (tid == 0) {                                // (what does not fit gives it back)
        sh_first = atomicAdd(g.used, n_stages);
        if (sh_first + n_stages > g.room) {
            atomicSub(g.used, n_stages);
            sh_first = -1;
        }
    }
    __syncthreads();
    const int first = sh_first;
    if (first < 0) return none();
    auto write = [&](int cell, int local, int y) {
        const int x0 = sh_cell[cell], k = x0 / RS, d = x0 % RS + 1, l = (int)(((int64_t)y * inv) >> 20), i = k + l, q = y - l * S;
        const uint32_t at = (uint32_t)((k * K + i) * SP + q);
        const int to_cell = i == K - 1 ? 0 : id[(i + 1) * RS + d - sh_size[q] - 1];
        g.stages[first + sh_at[cell] + local] = make_int4(ft.least[at], graph_label_bytes(cell, to_cell), (1 << 24) + (local << 11 | to_cell),
                                                          k << 22 | i << 14 | q << 8 | ft.run[at]);
    };
    if (n_stages <= list_room)
        for (int e = tid; e < n_stages; e += GRAPH_THREADS) write((int)(listed[e] >> 14), listed_at[e], (int)(listed[e] & 0x3fff));
    if (n_stages > list_room) {
        int *const counts = (int *)listed;             // (the list is of no use, and has room for GRAPH_CELLS: see launch_sparse_graph)
        for (int x = tid; x < n_cells; x += GRAPH_THREADS) counts[x] = 0;
        __syncthreads();
        stages(counts, [&](int cell, int n, uint64_t lanes, bool ok, int y) {
            if (ok) write(cell, n + __popcll(lanes & ((1ull << lane) - 1)), y);
        });
    }
    for (int x = tid; x < n_cells; x += GRAPH_THREADS) g.cells[j * GRAPH_CELLS + x] = sh_at[x];
    // chunks: a thread per first layer, r = K - 1 - k
    auto row_start = [&](int r) {                  // where the stages that begin with layer K - 1 - r start
        int lo = 1, hi = n_cells;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sh_cell[mid] / RS <= K - 1 - r) hi = mid; else lo = mid + 1;
        }
        return r >= K ? n_stages : sh_at[lo];
    };
    const int from = tid < K ? row_start(tid) : 0, to = tid < K ? row_start(tid + 1) : 0;
    int n_chunks;
    at = graph_scan((to - from + WAVE - 1) / WAVE, sh_scan, n_chunks);
    int32_t *const chunks = g.chunks + j * GRAPH_CHUNKS;
    for (int e = from; e < to; e += WAVE) chunks[at++] = e;
    if (tid == 0) chunks[n_chunks] = n_stages;
    // Where no plan is known, the latencies as they are may admit none up to some t_max: the lowest one with a plan, by as many
    // tries at a time as there are waves with room.  (With the fewest stages a cell has whatever can be had from it.)
    int32_t from_c = 0;
    if (U == INT32_MAX && n_stages <= GRAPH_SEARCH) {
        __syncthreads();                               // (the graph is there, and Q no longer needed)
        const int tries = min(FRONT_WAVES, (K * RS * 6 + list_room * 6) / 4 / n_cells);
        int32_t *const fewest = lds + wid * n_cells;
        const int4 *const all = g.stages + first;
        int32_t lo = max(low + 1, feasible), hi = c + 1;       // the answer is in [lo, hi], hi: none in the interval
        while (lo < hi) {                              // (uniform)
            const int32_t step = max(1, (hi - lo) / tries), x = lo + step * wid;
            if (tid == 0) sh_first = INT32_MAX;
            __syncthreads();
            if (wid < tries && x < hi) {
                for (int y = lane; y < n_cells; y += WAVE) fewest[y] = y == 0 ? 0 : 1 << 20;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                int4 w[4];                         // of chunks, as they are asked for
                int count[4], starts = 0, ends = 0;        // (a lane for each of 64 chunks, as in sparse_eval_kernel: a read in turn before each is
                                                   // 0.5 us a chunk)
                auto load = [&](int ch, int u) {
                    if ((ch & (WAVE - 1)) == 0) {
                        starts = chunks[min(ch + lane, n_chunks)];
                        ends = chunks[min(ch + lane + 1, n_chunks)];
                    }
                    const int e = __builtin_amdgcn_readlane(starts, ch & (WAVE - 1));
                    count[u] = __builtin_amdgcn_readlane(ends, ch & (WAVE - 1)) - e;
                    w[u] = all[e + lane];          // (there is room behind the last)
                };
#pragma unroll
                for (int u = 0; u < 4; ++u) load(u, u);
                for (int ch = 0; ch < n_chunks; ch += 4) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int4 v = w[u];
                        const bool in = lane < count[u];
                        load(ch + u + 4, u);
                        const int s = in ? *(const int32_t *)((const char *)fewest + ((uint32_t)v.y >> 17)) + 1 : 1 << 20;
                        int32_t t = v.x;
                        if (s > (v.w & 255))
                            t = s <= min(K, D) ? table[(((size_t)(s - 1) * K + (v.w >> 22)) * K + (v.w >> 14 & 255)) * S + (v.w >> 8 & 63)] : INF_I32;
                        if (t <= x) atomicMin((int32_t *)((char *)fewest + ((v.y & 0xffff) >> 1)), s);
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                    }
                }
                if (lane == 0 && fewest[n_cells - 1] < 1 << 20) atomicMin(&sh_first, x);
            }
            __syncthreads();
            const int32_t found = sh_first;            // the lowest try with a plan
            __syncthreads();
            if (found == INT32_MAX) lo = min(hi, lo + step * (min(tries, (hi - lo + step - 1) / step) - 1) + 1);
            else {
                hi = found;
                lo = max(lo, found - step + 1);
            }
        }
        from_c = lo;
    }
    if (tid == 0) g.heads[j] = GraphHead{first, n_stages, n_cells, n_chunks, from_c, n_stages > list_room};
}

// A workgroup for each interval; see band_bounds.
template <int W>
__global__ __launch_bounds__(GRAPH_THREADS) void sparse_graph_kernel(FrontTable ft, const int32_t *__restrict__ table, BandShapes bs, Problem p,
                                                                     int32_t max_finite, const int32_t *__restrict__ fronts,
                                                                     const int32_t *__restrict__ backs, const int32_t *__restrict__ totals,
                                                                     int32_t *plans, const int32_t *__restrict__ falls, GraphTable g, int list_room,
                                                                     int32_t *__restrict__ bounds, int once, int32_t *there)
{
    if (once && *there) return;
    sparse_graph<W>(blockIdx.x, ft, table, bs, p.K, p.D, max_finite, fronts, backs, totals, plans, falls, g, list_room);
    __syncthreads();
    band_bounds(p, max_finite, table, bs, fronts, WAVE * W, totals, plans, bounds, there, blockIdx.x);
}

struct SparseArgs {
    Problem p;
    const int32_t *table;
    GraphTable g;
    int32_t max_finite;
    const int32_t *cand, *list, *n_list_p;
    int32_t *Fmin, *Sbest;
    SparseOut o;
    int64_t *chunk_min;
    int prune, descending;
    unsigned long long *wave_relax;
};

// Listed candidates, a wave each.  A cell's label: sum << 32 | stages << 24 | number of its stage among the cell's << 11 | the cell
// behind.  Bound by the chain of chunks: a read of the label behind, two dozen instructions and a minimum in LDS each.  4096 candidates,
// 64 layers on 8 x 8: 65 us (the recurrence of some 600 of them, in two rounds, 224, and 97 for the plan); 1024, 64 on 16 x 8: 61
// (211, 84); 1024, 128 layers 64, and 95 for what has no graph (633, 172).
constexpr int SPARSE_WAVES = 4;
template <bool COUNT>
__global__ __launch_bounds__(SPARSE_WAVES * WAVE) void sparse_eval_kernel(SparseArgs a)
{
    __shared__ unsigned long long labels[SPARSE_WAVES][GRAPH_CELLS];
    __shared__ int sh_left[SPARSE_WAVES], sh_at;
    const int lane = threadIdx.x & (WAVE - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned long long *const L = labels[wid];
    char *const Lb = (char *)L;
    const int K = a.p.K, S = a.p.S, n = __builtin_amdgcn_readfirstlane(*a.n_list_p);
    const int32_t thr_lo = band_threshold(a.max_finite, min(lane, BAND_THRESHOLDS - 1));
    const int32_t thr_hi = band_threshold(a.max_finite, min(lane + WAVE, BAND_THRESHOLDS - 1));
    unsigned long long relaxed = 0;
    // candidates that are left to the recurrence, a lane each, listed by the workgroup (4096 additions to one word take 45 us)
    int left = 0, left_j = 0;
    auto list_left = [&](int at) {
        if (lane < left) a.o.todo[at + lane] = left_j;
        left = 0;
    };
    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); };    // (LDS takes a wave's accesses in order)
    for (int tk = blockIdx.x * SPARSE_WAVES + wid; tk < n; tk += gridDim.x * SPARSE_WAVES) {
        const int j = __builtin_amdgcn_readfirstlane(a.list[a.descending ? n - 1 - tk : tk]);
        const int32_t c_given = __builtin_amdgcn_readfirstlane(a.cand[j]), c = min(c_given, DEV_INF - 1);
        // the lowest threshold that is not below the candidate (they descend; the first has no filter)
        const int thr = max(0, min((int)(__popcll(__ballot(thr_lo >= c)) + __popcll(__ballot(lane + WAVE < BAND_THRESHOLDS && thr_hi >= c))), BAND_THRESHOLDS) - 1);
        const GraphHead h = a.g.heads[thr];
        const int n_stages = __builtin_amdgcn_readfirstlane(h.n_stages), n_cells = __builtin_amdgcn_readfirstlane(h.n_cells);
        const int n_chunks = __builtin_amdgcn_readfirstlane(h.n_chunks), first = __builtin_amdgcn_readfirstlane(h.first);
        const int4 *const stages = a.g.stages + first;
        const int32_t *const chunks = a.g.chunks + thr * GRAPH_CHUNKS;
        bool left_out = false;
        // one pass: `real`: only stages as they are
        auto pass = [&](bool real) {
            for (int x = lane; x < n_cells; x += WAVE) L[x] = x == 0 ? 0ull : ~0ull;
            fence();
            constexpr int AHEAD = 4;
            int4 w[AHEAD];
            int starts = 0, ends = 0;              // of chunks x0 .. x0 + 63, a lane each
            auto bounds = [&](int x) {
                if ((x & (WAVE - 1)) == 0) {
                    starts = chunks[min(x + lane, n_chunks)];
                    ends = chunks[min(x + lane + 1, n_chunks)];
                }
            };
            int count[AHEAD];
            auto load = [&](int x, int y) {
                bounds(x);
                const int from = __builtin_amdgcn_readlane(starts, x & (WAVE - 1));
                count[y] = x < n_chunks ? __builtin_amdgcn_readlane(ends, x & (WAVE - 1)) - from : 0;
                w[y] = stages[from + lane];        // (there is room behind the last)
            };
#pragma unroll
            for (int y = 0; y < AHEAD; ++y) load(y, y);
            for (int x = 0; x < n_chunks; x += AHEAD) {
#pragma unroll
                for (int y = 0; y < AHEAD; ++y) {
                    const int4 v = w[y];
                    const bool in = lane < count[y];
                    load(x + y + AHEAD, y);
                    const uint2 b = *(const uint2 *)(Lb + graph_label_behind(v.y, in));
                    const bool ok = in && v.x <= c && b.y != ~0u, as_is = b.x >> 24 < (uint32_t)(v.w & 255);
                    left_out |= ok && !as_is;
                    if (ok && (as_is || !real)) {
                        const unsigned long long own = (unsigned long long)(b.y + (uint32_t)v.x) << 32 | ((b.x & 0xff000000u) + (uint32_t)v.z);
                        __hip_atomic_fetch_min((unsigned long long *)(Lb + (v.y & 0xffff)), own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    fence();
                }
            }
            if (COUNT) relaxed += n_chunks;
        };
        auto label = [&](int cell) {               // (of all lanes the same)
            const unsigned long long v = L[cell];
            return (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        };
        bool settled = false;
        int32_t F = DEV_INF;
        int s = 0, slot = -1, route = ROUTE_PASS;
        if (n_stages >= 0 && c < __builtin_amdgcn_readfirstlane(h.from)) {
            settled = true;
            route = ROUTE_BELOW;
        } else if (n_stages >= 0) {
            pass(true);
            const unsigned long long root = label(n_cells - 1);
            if (root != ~0ull) {
                F = (int32_t)(root >> 32);
                s = (int)(root >> 24) & 255;
                if (lane == 0) slot = atomicAdd(a.o.n_slots, 1);
                slot = __builtin_amdgcn_readfirstlane(slot);
                if (slot >= SPARSE_PLANS) slot = -1;
                if (slot >= 0) {                   // the plan, from its first stage on
                    uint16_t *const plan = a.o.plans + (size_t)slot * K;
                    int cell = n_cells - 1;
                    for (int x0 = 0; x0 < s; x0 += WAVE) {
                        int own = 0;
                        for (int x = x0; x < min(s, x0 + WAVE); ++x) {
                            const uint32_t v = (uint32_t)label(cell);
                            own = lane == x - x0 ? (int)(v >> 11 & 0x1fff) | cell << 16 : own;
                            cell = v & 0x7ff;
                        }
                        if (x0 + lane < s) plan[x0 + lane] = (uint16_t)(a.g.cells[thr * GRAPH_CELLS + (own >> 16)] + (own & 0xffff));
                    }
                    if (lane == 0) a.o.plan_from[slot] = first;
                }
            }
            settled = true;
            if (__ballot(left_out) != 0) {
                pass(false);
                settled = label(n_cells - 1) >> 32 == root >> 32;
                route = ROUTE_SECOND_PASS;
            }
            if (!settled && n_stages <= GRAPH_LAYERS) {
                // Eq. 3 on the graph: layers of sums, by the number of stages
                int32_t *now = (int32_t *)L, *behind = now + n_cells;
                for (int x = lane; x < n_cells; x += WAVE) behind[x] = x == 0 ? 0 : DEV_INF;
                F = DEV_INF;
                s = 0;
                bool some = true;
                for (int layer = 1; layer <= a.p.Smax && some; ++layer) {
                    some = false;
                    for (int x = lane; x < n_cells; x += WAVE) now[x] = DEV_INF;
                    fence();
                    for (int x0 = 0; x0 < n_stages; x0 += WAVE) {
                        const int4 v = stages[x0 + lane];
                        const int32_t f = x0 + lane < n_stages ? *(const int32_t *)((const char *)behind + ((uint32_t)v.y >> 17)) : DEV_INF;
                        int32_t t = v.x;
                        if (f < DEV_INF && layer > (v.w & 255))        // no longer its least latency
                            t = a.table[(((size_t)(layer - 1) * K + (v.w >> 22)) * K + (v.w >> 14 & 255)) * S + (v.w >> 8 & 63)];
                        const bool ok = f < DEV_INF && t <= c;
                        if (ok) atomicMin((int32_t *)((char *)now + ((v.y & 0xffff) >> 1)), t + f);
                        some |= __ballot(ok) != 0;
                    }
                    fence();
                    const int32_t all = __builtin_amdgcn_readfirstlane(now[n_cells - 1]);
                    if (all < F) { F = all; s = layer; }
                    int32_t *const x = now;
                    now = behind;
                    behind = x;
                    if (COUNT) relaxed += (n_stages + WAVE - 1) / WAVE;
                }
                slot = -1;
                settled = true;
                route = ROUTE_LAYERS;
            }
        }
        if (COUNT && lane == 0) atomicAdd(&a.o.routes[settled ? route : ROUTE_LEFT], 1);
        if (lane == 0) {
            a.Fmin[j] = settled ? F : F_NOT_YET;
            a.Sbest[j] = settled ? s : 0;
            a.o.slot[j] = settled ? slot : -1;
            if (settled && a.prune && F < DEV_INF)
                atomicMin((long long *)&a.chunk_min[j / PRUNE_CHUNK], (long long)F + (long long)(a.p.B - 1) * c_given);
        }
        if (!settled) {
            left_j = lane == left ? j : left_j;
            if (++left == WAVE) {
                int at = 0;
                if (lane == 0) at = atomicAdd(a.o.n_todo, left);
                list_left(__builtin_amdgcn_readfirstlane(at));
            }
        }
    }
    if (lane == 0) sh_left[wid] = left;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < SPARSE_WAVES; ++w) {
        before += w < wid ? sh_left[w] : 0;
        all += sh_left[w];
    }
    if (threadIdx.x == 0 && all > 0) sh_at = atomicAdd(a.o.n_todo, all);
    __syncthreads();
    list_left(sh_at + before);
    if (COUNT) atomicAdd(a.wave_relax, lane == 0 ? relaxed : 0ull);
}

// the stages of the graphs, for the selection's plans
const int4 *graph_stages(int32_t *graph, int K, int D) { return graph_table(graph, K, D).stages; }

hipError_t launch_sparse_graph(hipStream_t st, const int32_t *table, const BandShapes &b, const Problem &p, int32_t max_finite,
                               const int32_t *work, const int32_t *front, const int32_t *fronts, const int32_t *backs,
                               const int32_t *totals, int32_t *plans, const int32_t *falls, int32_t *graph, int32_t *bounds, int32_t *there, bool once)
{
    const int K = p.K, D = p.D, RS = D <= 64 ? 64 : D <= 128 ? 128 : 256;
    const size_t cells = (size_t)K * RS * 6;       // (a multiple of 16)
    const size_t lds = std::max({front_lds_bytes(K, D, b.S), cells, std::min(cells + 6 * GRAPH_STAGES, (size_t)GRAPH_LDS)});
    const int list_room = (int)std::min((lds - cells) / 6, (size_t)GRAPH_STAGES);
    const auto kernel = D > 128 ? sparse_graph_kernel<4> : D > 64 ? sparse_graph_kernel<2> : sparse_graph_kernel<1>;
    if (lds > 48 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(BAND_THRESHOLDS), dim3(GRAPH_THREADS), lds, st, front_table(work, front, K, b.S, b.sizes, false),
                       table, b, p, max_finite, fronts, backs, totals, plans, falls, graph_table(graph, K, D), list_room, bounds, once ? 1 : 0, there);
    return hipGetLastError();
}

hipError_t launch_sparse_eval(hipStream_t st, const FastArgs &f, const int32_t *table, int32_t *graph, int32_t max_finite, const SparseOut &o, bool count,
                              int most, int n_cu)
{
    SparseArgs a{f.p, table, graph_table(graph, f.p.K, f.p.D), max_finite, f.cand, f.list, f.n_list_p, f.Fmin, f.Sbest, o, f.chunk_min,
                 f.prune, f.descending, f.wave_relax};
    const auto kernel = count ? sparse_eval_kernel<true> : sparse_eval_kernel<false>;
    const int grid = std::max(1, std::min((most + SPARSE_WAVES - 1) / SPARSE_WAVES, 3 * n_cu));     // (three fit a compute unit's LDS)
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(SPARSE_WAVES * WAVE), 0, st, a);
    return hipGetLastError();
}

}  // namespace alpa
