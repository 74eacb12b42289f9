// Host-side test driver: the library's own host code over a HIP runtime that is made up here.  The
// executable defines every HIP function that libalpa_dp.so imports, so no GPU and no driver is touched
// and no kernel runs: allocations are addresses in a reserved range that is never used twice, and a
// launch is its kernel's name and its pointer arguments.  That shows, on the CPU, what a call would have
// the GPU read and write: arguments that are null, or that lie in memory already given back.
//
//   g++ -std=c++17 -rdynamic -o driver tests/fake_hip_driver.cpp -Iinclude libalpa_dp.so
//   ./driver <scenario>          prints OK, or what is wrong (exit status 1)
#include "../include/alpa_dp.h"

#include <cxxabi.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

using Stream = void *;
struct Dim3 { uint32_t x, y, z; };
constexpr int OK = 0, INVALID = 1, OUT_OF_MEMORY = 2, CAPTURE_UNSUPPORTED = 900, CAPTURE_IMPLICIT = 906;
constexpr int D2H = 2, MODE_GLOBAL = 0, MODE_RELAXED = 2;

struct Block { size_t bytes; bool live; };
struct Launch { std::string kernel; std::vector<std::pair<uintptr_t, std::string>> pointers; };

struct Runtime {
    uintptr_t base = 0, next = 0;
    std::map<uintptr_t, Block> blocks;             // by first address
    std::map<const void *, std::string> kernels;   // host stub -> demangled name
    std::vector<Launch> launches;
    bool capturing = false;
    int mode = MODE_GLOBAL, last_error = OK;
    int waits_for_capture = 0;                     // synchronisation, allocation or release in a capture
    int mallocs = 0, syncs = 0;
    int fail_from = 0, fail_to = 0, failed = 0;    // the allocations [from, to) fail
    int32_t n_distinct = 100, largest = 5000, falls = 0;      // what the kernels would have found in the table
    Dim3 grid{}, block{};
    size_t shared = 0;
    Stream stream = nullptr;
};
static Runtime &rt()
{
    static Runtime r;
    if (!r.base) {
        r.base = (uintptr_t)mmap(nullptr, 1ull << 40, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        r.next = r.base;
    }
    return r;
}
static const Block *block_of(uintptr_t p)
{
    auto it = rt().blocks.upper_bound(p);
    if (it == rt().blocks.begin()) return nullptr;
    --it;
    return p < it->first + it->second.bytes ? &it->second : nullptr;
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *)
{
    int status = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    rt().kernels[stub] = d ? d : name;
    free(d);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, Stream st)
{
    rt().grid = grid; rt().block = block; rt().shared = shared; rt().stream = st;
    return OK;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, Stream *st)
{
    *grid = rt().grid; *block = rt().block; *shared = rt().shared; *st = rt().stream;
    return OK;
}
int hipLaunchKernel(const void *stub, Dim3, Dim3, void **args, size_t, Stream)
{
    const std::string &sig = rt().kernels[stub];
    Launch l;
    const size_t open = sig.rfind('(');
    l.kernel = sig.substr(0, open);
    std::string params = sig.substr(open + 1, sig.size() - open - 2);
    for (size_t n = 0, at = 0; at <= params.size(); ++n) {
        size_t comma = params.find(',', at);
        if (comma == std::string::npos) comma = params.size();
        const std::string type = params.substr(at, comma - at);
        if (type.find('*') != std::string::npos) l.pointers.push_back({*(uintptr_t *)args[n], type});
        at = comma + 1;
    }
    rt().launches.push_back(l);
    return OK;
}
int hipMalloc(void **p, size_t bytes)
{
    if (rt().capturing && rt().mode != MODE_RELAXED) { ++rt().waits_for_capture; return CAPTURE_UNSUPPORTED; }
    const int n = rt().mallocs++;
    if (n >= rt().fail_from && n < rt().fail_to) { ++rt().failed; *p = nullptr; return rt().last_error = OUT_OF_MEMORY; }
    *p = (void *)rt().next;
    rt().blocks[rt().next] = {bytes, true};
    rt().next += (bytes + 4096) & ~(size_t)4095;
    return OK;
}
int hipFree(void *p)
{
    if (!p) return OK;
    if (rt().capturing) { ++rt().waits_for_capture; return CAPTURE_UNSUPPORTED; }
    auto it = rt().blocks.find((uintptr_t)p);
    if (it == rt().blocks.end() || !it->second.live) { printf("release of something that is not allocated\n"); exit(1); }
    it->second.live = false;
    return OK;
}
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, Stream)
{
    Launch l{"memcpy", {}};
    for (const void *p : {(const void *)dst, src})
        if (block_of((uintptr_t)p)) l.pointers.push_back({(uintptr_t)p, "void*"});
    rt().launches.push_back(l);
    if (kind != D2H) return OK;
    memset(dst, 0, bytes);
    if (bytes == 4) memcpy(dst, &rt().n_distinct, 4);
    if (bytes == 12) ((int32_t *)dst)[1] = rt().largest;       // (smallest, largest, does one fall)
    if (bytes == 12) ((int32_t *)dst)[2] = rt().falls;
    return OK;
}
int hipMemsetAsync(void *, int, size_t, Stream) { return OK; }
int hipStreamSynchronize(Stream)
{
    if (rt().capturing) { ++rt().waits_for_capture; return CAPTURE_UNSUPPORTED; }
    ++rt().syncs;
    return OK;
}
int hipStreamIsCapturing(Stream st, int *status)
{
    *status = st && rt().capturing ? 1 : 0;
    return !st && rt().capturing ? CAPTURE_IMPLICIT : OK;
}
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipSetDevice(int) { return OK; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return OK; }
int hipEventCreate(void **e) { *e = e; return OK; }
int hipEventDestroy(void *) { return OK; }
int hipEventRecord(void *, Stream) { return OK; }
int hipEventSynchronize(void *) { return OK; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1; return OK; }
int hipFuncSetAttribute(const void *, int, int) { return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 8; return OK; }
int hipGetLastError(void) { const int e = rt().last_error; rt().last_error = OK; return e; }
int hipThreadExchangeStreamCaptureMode(int *mode) { std::swap(rt().mode, *mode); return OK; }
const char *hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }
int hipGetSymbolAddress(void **, const void *) { return INVALID; }
int hipGetDevicePropertiesR0600(void *, int) { return INVALID; }
}

// from the next allocation but `skip` on, `n` of them fail
static void fail_mallocs(int skip, int n)
{
    rt().fail_from = rt().mallocs + skip;
    rt().fail_to = rt().fail_from + n;
    rt().failed = 0;
}

static int bad = 0;
#define CHECK(cond, ...) do { if (!(cond)) { printf(__VA_ARGS__); printf(" [%s]\n", #cond); ++bad; } } while (0)

// Every pointer of the launches from number `from` on lies in memory that is allocated now.
static void check_launches(size_t from, size_t to, const char *what)
{
    for (size_t n = from; n < to; ++n) {
        const Launch &l = rt().launches[n];
        for (auto &[p, type] : l.pointers) {
            const Block *b = block_of(p);
            if (b) CHECK(b->live, "%s: %s: a %s in memory that was given back", what, l.kernel.c_str(), type.c_str());
            // the work areas of the candidate list are never optional
            else if (l.kernel.find("bitmap_") != std::string::npos || l.kernel.find("radix_") != std::string::npos ||
                     l.kernel.find("gather_") != std::string::npos)
                CHECK(p != 0, "%s: %s: a %s is null", what, l.kernel.c_str(), type.c_str());
        }
    }
}

// `repeat`: fill the list up to so many shapes with the first one; negative: only so many shapes
static alpa_dp_t *create_problem(int K, int N, int M, int repeat = 0)
{
    std::vector<alpa_shape_t> shapes;
    for (int m = 1; m <= M; m *= 2) shapes.push_back({1, m});
    for (int n = 2; n <= N; ++n) shapes.push_back({n, M});
    while ((int)shapes.size() < repeat) shapes.push_back(shapes[0]);
    if (repeat < 0) shapes.resize(-repeat);
    alpa_dp_t *h = nullptr;
    static const int32_t table = 7;                // (nothing reads it)
    const int rc = alpa_dp_create(&h, &table, K, N, M, 8, shapes.data(), (int)shapes.size());
    if (rc) { printf("create: %d %s\n", rc, alpa_dp_last_error()); exit(1); }
    CHECK(alpa_dp_set_stream(h, (void *)0x1000) == 0, "stream");   // (the null stream cannot be recorded)
    return h;
}
// 12 layers on 2 x 8: 12 * 78 * 5 = 4680 table entries, 100 distinct values of up to 5000
constexpr int K = 12, N = 2, M = 8, ENTRIES = K * (K * (K + 1) / 2) * 5;
static alpa_dp_t *create() { return create_problem(K, N, M); }
static void *device_array(size_t bytes) { void *p; hipMalloc(&p, bytes); return p; }

// a reported ENOMEM leaves a handle that works, or says ENOMEM again
static void out_of_memory()
{
    for (int big : {0, 1}) {                       // values for the bitmap, and for the sort
        rt().largest = big ? 1 << 24 : 5000;
        for (int nth = 0; nth < 2; ++nth) {
            alpa_dp_t *h = create();
            std::vector<int32_t> list(3 * ENTRIES, 9);
            alpa_plan_t plan;
            fail_mallocs(nth, 9);
            const int rc = alpa_dp_solve(h, list.data(), (int)list.size(), 0, nullptr, &plan);
            const bool failed = rt().failed > 0;
            fail_mallocs(0, 0);
            CHECK(rc == (failed ? ALPA_DP_ENOMEM : 0), "long list, allocation %d fails: %d", nth, rc);
            const size_t from = rt().launches.size();
            CHECK(alpa_dp_solve(h, nullptr, 0, 0, nullptr, &plan) == 0, "solve after it");
            CHECK(alpa_dp_restrict_equal_layers(h) == 0, "restriction after it");
            CHECK(alpa_dp_best(h, &plan) == 0, "best after it");
            check_launches(from, rt().launches.size(), "after a failed allocation");
            // the same with the restriction first
            fail_mallocs(nth, 9);
            (void)alpa_dp_solve(h, list.data(), (int)list.size(), 0, nullptr, &plan);
            fail_mallocs(0, 0);
            const size_t next = rt().launches.size();
            CHECK(alpa_dp_restrict_equal_layers(h) == 0, "restriction after a second one");
            check_launches(next, rt().launches.size(), "restriction after a failed allocation");
            alpa_dp_destroy(h);
        }
    }
}

// a solve on device pointers with a list of up to as many values as the table has entries only queues work:
// no allocation, no wait, also recorded into a graph as the handle's first call
static void ordinary_lists()
{
    for (int sort : {0, 1})
        for (int n : {0, 1025, 2000, ENTRIES}) {
            for (int capture : {1, 0}) {
                alpa_dp_t *h = create();
                CHECK(alpa_dp_set_tuning(h, ALPA_DP_TUNE_DISTINCT_BY_SORT, sort) == 0, "tuning");
                auto *d_list = (int32_t *)device_array((size_t)ENTRIES * 4);
                auto *d_T = (int64_t *)device_array((size_t)ENTRIES * 8);
                rt().capturing = capture;
                rt().waits_for_capture = rt().mallocs = rt().syncs = 0;
                const size_t from = rt().launches.size();
                const int rc = alpa_dp_solve_dev(h, n ? d_list : nullptr, n, 0, d_T, nullptr);
                rt().capturing = false;
                CHECK(rc == 0, "list of %d, sort %d, capture %d: %d (%s)", n, sort, capture, rc, alpa_dp_last_error());
                CHECK(rt().waits_for_capture + rt().mallocs + rt().syncs == 0,
                      "list of %d, sort %d, capture %d: %d allocations, %d waits, %d of them in the capture", n, sort,
                      capture, rt().mallocs, rt().syncs, rt().waits_for_capture);
                check_launches(from, rt().launches.size(), "ordinary list");
                alpa_dp_destroy(h);
            }
        }
}

static size_t live_bytes()
{
    size_t n = 0;
    for (auto &b : rt().blocks) n += b.second.live ? b.second.bytes : 0;
    return n;
}

// a graph's kernels keep their memory, whatever the handle is asked for afterwards
static void recorded_solve()
{
    const size_t before = live_bytes();
    alpa_dp_t *h = create();
    std::vector<int32_t> list(200 * ENTRIES, 9);
    alpa_plan_t plan;
    auto eager = [&](int n) { return alpa_dp_solve(h, list.data(), n, 0, nullptr, &plan); };
    const size_t at_first = live_bytes();
    const size_t from = rt().launches.size();
    rt().capturing = true;
    CHECK(alpa_dp_solve_dev(h, nullptr, 0, 0, nullptr, nullptr) == 0, "recorded solve: %s", alpa_dp_last_error());
    rt().capturing = false;
    const size_t to = rt().launches.size();
    for (int n : {2, 5, 6, 9, 17, 18, 40}) {
        const size_t mine = rt().launches.size();
        CHECK(eager(n * ENTRIES) == 0, "list of %d times the entries", n);
        check_launches(mine, rt().launches.size(), "eager solve");
        check_launches(from, to, "replay after a longer list");
    }
    // what has been outgrown is less than what is in use, and that at most twice the longest list
    CHECK(live_bytes() - at_first < (size_t)2 * 2 * 40 * ENTRIES * 50, "%zu bytes held", live_bytes() - at_first);
    fail_mallocs(0, 9);
    CHECK(eager(200 * ENTRIES) == ALPA_DP_ENOMEM, "no room");
    fail_mallocs(0, 0);
    check_launches(from, to, "replay after a failed attempt");
    const size_t mine = rt().launches.size();
    CHECK(eager(40 * ENTRIES) == 0, "list that has found room before");
    check_launches(mine, rt().launches.size(), "eager solve after a failed attempt");
    alpa_dp_destroy(h);
    CHECK(live_bytes() == before, "%zu bytes left by destroy", live_bytes() - before);
}

// a list of any length only queues work on the caller's stream, recorded or not: the arrays grow without a wait
static void long_lists()
{
    for (int capture : {1, 0}) {
        alpa_dp_t *h = create();
        auto *d_list = (int32_t *)device_array((size_t)100 * ENTRIES * 4);
        auto *d_T = (int64_t *)device_array((size_t)100 * ENTRIES * 8);
        rt().capturing = capture;
        rt().waits_for_capture = rt().syncs = 0;
        const size_t from = rt().launches.size();
        for (int n : {1, 10, 100, 2}) {
            const int rc = alpa_dp_solve_dev(h, d_list, n * ENTRIES, 0, d_T, nullptr);
            CHECK(rc == 0, "list of %d times the entries, capture %d: %d (%s)", n, capture, rc, alpa_dp_last_error());
        }
        rt().capturing = false;
        CHECK(rt().waits_for_capture + rt().syncs == 0, "capture %d: %d waits, %d in the capture", capture, rt().syncs,
              rt().waits_for_capture);
        check_launches(from, rt().launches.size(), "long lists");
        CHECK(rt().mode == MODE_GLOBAL, "the thread's capture mode is left changed");
        alpa_dp_destroy(h);
    }
}

// times are those of a solve that has run: none are there behind one that was only recorded
static void timing()
{
    alpa_dp_t *h = create();
    alpa_plan_t plan;
    float a, b, c;
    CHECK(alpa_dp_last_timing(h, &a, &b, &c) == ALPA_DP_EINVAL, "times of no solve");
    const int32_t Bs[] = {1, 3};
    alpa_plan_t plans[2];
    for (int eager = 0; eager < 3; ++eager) {
        rt().capturing = true;
        CHECK(alpa_dp_solve_dev(h, nullptr, 0, 0, nullptr, nullptr) == 0, "recorded solve");
        rt().capturing = false;
        CHECK(alpa_dp_last_timing(h, &a, &b, &c) == ALPA_DP_EHIP, "times of a solve that was recorded");
        const int rc = eager == 2 ? alpa_dp_solve_sweep(h, nullptr, 0, 0, Bs, 2, plans) : alpa_dp_solve(h, nullptr, 0, 0, nullptr, &plan);
        CHECK(rc == 0 && alpa_dp_last_timing(h, &a, &b, &c) == 0, "times of a solve: %s", alpa_dp_last_error());
    }
    alpa_dp_destroy(h);
}

// memory too short for old and new arrays together: without a graph the old ones make room
static void short_memory()
{
    alpa_dp_t *h = create();
    std::vector<int32_t> list(9 * ENTRIES, 9);
    alpa_plan_t plan;
    for (int nth : {0, 1}) {
        fail_mallocs(nth, 1);
        const size_t from = rt().launches.size();
        CHECK(alpa_dp_solve(h, list.data(), (4 + 5 * nth) * ENTRIES, 0, nullptr, &plan) == 0, "allocation %d fails: %s",
              nth, alpa_dp_last_error());
        fail_mallocs(0, 0);
        check_launches(from, rt().launches.size(), "solve in short memory");
    }
    alpa_dp_destroy(h);
}

// which kernels a solve of n quantiles (0: all 5000 values) launches, each name between blanks
static std::string kernels_of(alpa_dp_t *h, int n)
{
    const size_t from = rt().launches.size();
    CHECK(alpa_dp_solve_dev(h, nullptr, n, 0, (int64_t *)device_array(8 * 5000), nullptr) == 0, "solve");
    std::string all = " ";
    for (size_t x = from; x < rt().launches.size(); ++x) {
        std::string k = rt().launches[x].kernel;
        k.erase(0, k.rfind("alpa::") + 6);
        for (char c : k) if (c != ' ') all += c;
        all += " ";
    }
    return all;
}

// which form of the recurrence serves which sizes and lists, and when a table's bounds are computed
static void routes()
{
    rt().n_distinct = 5000;
    struct { int K, N, M, n; const char *has, *has_not; int repeat = 0; } cases[] = {
        // up to 8 devices: beyond two candidates per compute unit in lane groups, not with eight waves each
        {24, 1, 4, 1500, " recurrence_fast_kernel<2,1,1,false,false,false,true> ", "recurrence_fast_kernel<2,2,1,false"},
        {40, 2, 4, 2048, " recurrence_fast_kernel<3,1,1,false,false,false,true> ", "recurrence_fast_kernel<3,2,1,false"},
        {64, 1, 2, 600, " recurrence_fast_kernel<4,1,1,false,false,false,true> ", "recurrence_fast_kernel<4,2,1,false"},
        {64, 1, 2, 512, " recurrence_fast_kernel<4,4,1,false,false,false,false> ", "false,true> "},
        {72, 1, 2, 2048, " recurrence_fast_kernel<5,1,1,false,false,false,true> ", "recurrence_band"},
        {128, 1, 2, 2048, " recurrence_fast_kernel<8,1,1,false,false,false,true> ", "recurrence_band"},
        {96, 1, 4, 2048, " recurrence_fast_kernel<6,1,1,false,false,false,true> ", "recurrence_band"},
        {97, 3, 1, 2048, " recurrence_fast_kernel<7,1,1,false,false,false,true> ", "recurrence_band"},
        // a workgroup per candidate: on more than 4 devices from 65 layers on, on more than 8, and where the layers fit in LDS
        {24, 3, 4, 1500, " recurrence_band_kernel<64,4,false,false> ", "recurrence_fast"},
        {64, 8, 8, 1500, " recurrence_band_kernel<64,4,false,false> ", "recurrence_fast"},
        {65, 5, 1, 2048, " recurrence_band_kernel<64,8,false,false> ", "recurrence_fast"},
        {72, 2, 4, 2048, " recurrence_band_kernel<64,8,false,false> ", "recurrence_fast"},
        {129, 1, 2, 300, " recurrence_band_kernel<64,0,false,false> ", "recurrence_generic"},
        {139, 8, 8, 300, " recurrence_band_kernel<64,0,false,false> ", "recurrence_generic"},
        {100, 64, 1, 300, " recurrence_band_kernel<64,8,false,false> ", "recurrence_fast"},
        {86, 16, 8, 300, " recurrence_band_kernel<128,0,false,false> ", "recurrence_fast"},
        {59, 32, 8, 300, " recurrence_band_kernel<256,0,false,false> ", "recurrence_generic"},
        {60, 32, 8, 300, " recurrence_generic_kernel ", "recurrence_band"},
        // repeated shapes are one to it
        {220, 1, 8, 300, " recurrence_band_kernel<64,0,false,false> ", "recurrence_generic", 64},
        {205, 14, 1, 300, " recurrence_band_kernel<64,0,false,false> ", "recurrence_generic", 64},
        {124, 16, 8, 300, " recurrence_fast_kernel<8,1,2,false,false,true,false> ", "recurrence_band"},
        {96, 110, 1, 300, " recurrence_fast_kernel<6,1,2,false,false,true,false> ", "recurrence_band", -64},
        {96, 110, 1, 7, " recurrence_fast_kernel<6,2,2,false,false,true,false> ", "recurrence_band", -64},
        {110, 49, 2, 300, " recurrence_fast_kernel<7,1,2,false,false,true,false> ", "recurrence_band"},
        {112, 63, 2, 7, " recurrence_fast_kernel<7,2,2,false,false,true,false> ", "recurrence_band"},
        {128, 28, 4, 300, " recurrence_fast_kernel<8,1,2,false,false,true,false> ", "recurrence_band"},
    };
    for (auto &c : cases) {
        alpa_dp_t *h = create_problem(c.K, c.N, c.M, c.repeat);
        (void)kernels_of(h, c.n);
        const std::string k = kernels_of(h, c.n);  // with the bounds
        CHECK(k.find(c.has) != std::string::npos, "%d layers on %dx%d, %d: no%sin%s", c.K, c.N, c.M, c.n, c.has, k.c_str());
        CHECK(k.find(c.has_not) == std::string::npos, "%d layers on %dx%d, %d: %s in%s", c.K, c.N, c.M, c.n, c.has_not,
              k.c_str());
        alpa_dp_destroy(h);
    }
    // graphs where the band kernel serves, no shape is repeated and no latency falls with the stages behind: made with the bounds (by
    // a kernel that makes none where one falls, but the bounds), gone through in each round in front of the recurrence; not behind a
    // restriction
    struct { int K, N, M, repeat, falls; bool makes, graphs; } graphs[] = {
        {24, 2, 8, 0, 0, true, true}, {24, 2, 8, 0, 1, true, false}, {24, 2, 8, 8, 0, false, false}, {24, 1, 8, 0, 0, false, false},
        {64, 16, 8, 0, 0, true, true}, {60, 32, 8, 0, 0, false, false}};
    for (auto &c : graphs) {
        rt().falls = c.falls;
        alpa_dp_t *h = create_problem(c.K, c.N, c.M, c.repeat);
        rt().falls = 0;
        for (int n : {0, 600}) {                   // (5000 values: two rounds)
            for (int solve = 0; solve < 2; ++solve) {
                const std::string k = kernels_of(h, n);
                int made = 0, gone = 0;
                for (size_t at = 0; (at = k.find(" sparse_graph_kernel<", at)) != std::string::npos; ++at) ++made;
                for (size_t at = 0; (at = k.find(" sparse_eval_kernel<false> recurrence_band_kernel<", at)) != std::string::npos; ++at) ++gone;
                CHECK(made == (c.makes && n == 0 && solve == 0) && gone == (c.graphs ? n == 0 ? 2 : 1 : 0),
                      "%d layers on %dx%d, %d, %d: %d made, %d gone through in%s", c.K, c.N, c.M, c.repeat, c.falls, made, gone, k.c_str());
            }
        }
        CHECK(alpa_dp_restrict_equal_layers(h) == 0, "restriction");
        CHECK(kernels_of(h, 0).find(" sparse_eval") == std::string::npos, "%d layers on %dx%d: graphs of stages of equal layers", c.K, c.N, c.M);
        alpa_dp_destroy(h);
    }
    // forms that the tuning call asks for, on the meshes of the register/LDS kernel
    struct { int K, N, M, n, key, value; const char *has; } tuned[] = {
        {64, 2, 4, 300, ALPA_DP_TUNE_LANE_GROUPS, 2, " recurrence_fast_kernel<4,1,1,false,false,false,true> "},
        {17, 5, 1, 300, ALPA_DP_TUNE_LANE_GROUPS, 64, " recurrence_fast_kernel<2,1,1,false,false,false,true> "},
        {128, 3, 1, 600, ALPA_DP_TUNE_LANE_GROUPS, 1, " recurrence_fast_kernel<8,1,1,false,false,false,false> "},
        {48, 5, 1, 301, ALPA_DP_TUNE_CANDIDATES_PER_WG, 2, " recurrence_fast_kernel<3,1,2,false,false,false,false> "},
        {128, 1, 4, 301, ALPA_DP_TUNE_CANDIDATES_PER_WG, 2, " recurrence_fast_kernel<8,1,2,false,false,false,false> "},
    };
    for (auto &c : tuned) {
        alpa_dp_t *h = create_problem(c.K, c.N, c.M);
        CHECK(alpa_dp_set_tuning(h, c.key, c.value) == 0, "tuning");
        const std::string k = kernels_of(h, c.n);
        CHECK(k.find(c.has) != std::string::npos, "%d layers on %dx%d, %d, key %d: no%sin%s", c.K, c.N, c.M, c.n, c.key, c.has, k.c_str());
        alpa_dp_destroy(h);
    }
    // bounds: by the first solve, or by the second; not recorded into a small problem's graph, but for the band kernel's (which replays
    // behind the first find there)
    struct { int K, N, M, n, by; } bounds[] = {{8, 1, 4, 0, 2}, {24, 2, 8, 1000, 1}, {40, 1, 8, 512, 2}, {64, 1, 2, 300, 2},
                                               {64, 2, 8, 12, 1}, {56, 4, 8, 130, 1}, {40, 8, 8, 12, 1}, {56, 8, 8, 12, 1},
                                               {26, 12, 16, 23, 1}, {6, 16, 8, 12, 1}, {64, 8, 8, 300, 1}, {48, 8, 8, 2000, 1}, {24, 8, 8, 5000, 1},
                                               {40, 1, 8, 2048, 1}, {50, 1, 8, 12, 1}};
    auto bounds_in = [](const std::string &k) {
        return k.find("bound_layer") != std::string::npos || k.find("band_thresholds") != std::string::npos;
    };
    for (auto &c : bounds) {
        alpa_dp_t *h = create_problem(c.K, c.N, c.M);
        rt().capturing = true;
        const bool recorded = bounds_in(kernels_of(h, c.n));
        rt().capturing = false;
        CHECK(recorded == (c.by == 1), "%d layers on %dx%d, %d: bounds in the graph: %d", c.K, c.N, c.M, c.n, recorded);
        alpa_dp_destroy(h);
        h = create_problem(c.K, c.N, c.M);
        const bool band = kernels_of(h, c.n).find("recurrence_band") != std::string::npos;
        alpa_dp_destroy(h);
        h = create_problem(c.K, c.N, c.M);
        for (int restricted = 0; restricted < 2; ++restricted) {
            for (int solve = 1; solve <= 3; ++solve) {
                const std::string kernels = kernels_of(h, c.n);
                const bool found = bounds_in(kernels), exact = kernels.find("band_exact_bounds") != std::string::npos;
                CHECK(exact == (band && solve == 2 && !restricted), "%d layers on %dx%d, %d: solve %d, exact bounds %d", c.K, c.N,
                      c.M, c.n, solve, exact);
                CHECK(found == (solve == c.by && !restricted), "%d layers on %dx%d, %d: solve %d, bounds %d", c.K, c.N, c.M,
                      c.n, solve, found);
            }
            const size_t from = rt().launches.size();
            CHECK(alpa_dp_restrict_equal_layers(h) == 0, "restriction");
            bool again = false;                    // (they are there: the restriction computes them anew)
            for (size_t x = from; x < rt().launches.size(); ++x)
                again |= bounds_in(rt().launches[x].kernel);
            CHECK(again, "%d layers on %dx%d: bounds of the old table", c.K, c.N, c.M);
        }
        alpa_dp_destroy(h);
    }
}

// a sweep keeps as many sets of layers as there is memory for, and needs none of its own
static void sweep_memory()
{
    const int values = 256;
    struct { int K, N, M; } cases[] = {{48, 32, 8}, {40, 8, 8}, {40, 1, 8}};
    for (auto &c : cases) {
        for (int failures : {0, 1, 3, 8, 40}) {
            alpa_dp_t *h = create_problem(c.K, c.N, c.M);
            std::vector<int32_t> B(values, 3);
            std::vector<alpa_plan_t> plans(values);
            const size_t before = live_bytes(), from = rt().launches.size();
            fail_mallocs(0, failures);
            const int rc = alpa_dp_solve_sweep(h, nullptr, 12, 0, B.data(), values, plans.data());
            fail_mallocs(0, 0);
            CHECK(rc == (failures <= 8 ? ALPA_DP_OK : ALPA_DP_ENOMEM), "%d layers on %dx%d, %d failures: %d", c.K, c.N, c.M, failures, rc);
            check_launches(from, rt().launches.size(), "sweep");
            int walks = 0;
            for (size_t x = from; x < rt().launches.size(); ++x) walks += rt().launches[x].kernel.find("plan_walk") != std::string::npos;
            // (half the sets at each failure; all 256 are below 1 GiB)
            CHECK(rc != 0 || walks == 1 << failures, "%d layers on %dx%d, %d failures: %d launches", c.K, c.N, c.M, failures, walks);
            CHECK(live_bytes() - before < 1ull << 30, "%zu bytes", live_bytes() - before);
            alpa_dp_destroy(h);
        }
    }
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "out_of_memory") out_of_memory();
    else if (what == "ordinary_lists") ordinary_lists();
    else if (what == "recorded_solve") recorded_solve();
    else if (what == "long_lists") long_lists();
    else if (what == "short_memory") short_memory();
    else if (what == "timing") timing();
    else if (what == "routes") routes();
    else if (what == "sweep_memory") sweep_memory();
    else { printf("unknown scenario\n"); return 1; }
    if (!bad) printf("OK\n");
    return bad ? 1 : 0;
}
