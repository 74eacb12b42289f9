// C ABI of the operator-clustering step: argument checks, device buffers, launch order.
#include "../../include/alpa_dp.h"
#include "internal.hpp"

#include <algorithm>
#include <memory>
#include <new>
#include <string>

using namespace alpa;

extern "C" __attribute__((visibility("hidden"))) int alpa_dp_set_error_(int code, const char *msg);   // alpa_dp_abi.hip

namespace {

struct DevBuf {                       // frees on scope exit
    void *p = nullptr;
    ~DevBuf() { if (p) (void)hipFree(p); }
    hipError_t alloc(size_t bytes) { return hipMalloc(&p, bytes ? bytes : 4); }
    template <class T> T *as() const { return (T *)p; }
};

int fail(int code, const std::string &msg) { return alpa_dp_set_error_(code, msg.c_str()); }

#define HIPCHK(expr)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(e_ == hipErrorOutOfMemory ? ALPA_DP_ENOMEM : ALPA_DP_EHIP,          \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                 \
    } while (0)

}  // namespace

static int cluster_layers_impl(const int32_t *flop, int K, const int32_t *edge_src,
                               const int32_t *edge_dst, const int64_t *edge_bytes, int num_edges,
                               int L, int delta_ppm, int64_t *out_comm, int64_t *out_sumsq,
                               int32_t *out_first_op, float *out_ms, int exact,
                               unsigned max_spins = CLUSTER_MAX_SPINS)
{
    if (!flop || !out_comm || !out_sumsq || !out_first_op)
        return fail(ALPA_DP_EINVAL, "null argument");
    if (K < 1 || K > ALPA_CLUSTER_MAX_OPS) return fail(ALPA_DP_EINVAL, "K out of range");
    if (L < 1 || L > ALPA_CLUSTER_MAX_OPS) return fail(ALPA_DP_EINVAL, "L out of range");
    if (num_edges < 0 || (num_edges > 0 && (!edge_src || !edge_dst || !edge_bytes)))
        return fail(ALPA_DP_EINVAL, "edge list is null or num_edges < 0");
    if (delta_ppm < 0 || delta_ppm > 1000000000) return fail(ALPA_DP_EINVAL, "delta_ppm out of range");
    int64_t total = 0;
    for (int k = 0; k < K; ++k) {
        if (flop[k] < 0) return fail(ALPA_DP_EINVAL, "negative FLOP figure");
        total += flop[k];
    }
    if (total >= (1ll << 31)) return fail(ALPA_DP_EOVERFLOW, "total FLOP >= 2^31");
    if (total * (int64_t)L >= (1ll << 42)) return fail(ALPA_DP_EOVERFLOW, "total FLOP * L >= 2^42");
    int64_t all_bytes = 0;
    for (int e = 0; e < num_edges; ++e) {
        if (edge_src[e] < 0 || edge_dst[e] >= K || edge_src[e] >= edge_dst[e])
            return fail(ALPA_DP_EINVAL, "edge must go from an earlier to a later operator");
        if (edge_bytes[e] < 0) return fail(ALPA_DP_EINVAL, "negative edge size");
        if (edge_bytes[e] >= (1ll << 62) - all_bytes)
            return fail(ALPA_DP_EOVERFLOW, "sum of edge sizes >= 2^62");
        all_bytes += edge_bytes[e];
    }
    // FLOP(i..n) * L * 10^6 <= (10^6 + delta_ppm) * total, for integers, is FLOP(i..n) <= cap
    const int64_t cap = ((1000000ll + delta_ppm) * total) / ((int64_t)L * 1000000ll);

    hipStream_t st = nullptr;
    // inputs, results and work memory are parts of one allocation (each costs tens of microseconds, and so does
    // its release); the edges go up in one copy, the results come down in one
    const size_t E = (size_t)num_edges;
    const int width = cluster_band_width(flop, K, cap);
    const size_t in64 = E + (2 * E + (size_t)K + 1) / 2, out64 = 3 + ((size_t)L + 2) / 2;
    DevBuf mem;
    HIPCHK(mem.alloc((in64 + out64 + cluster_work_i64(K, L, width)) * 8));
    std::unique_ptr<int64_t[]> stage(new (std::nothrow) int64_t[std::max(in64, out64)]);
    if (!stage) return fail(ALPA_DP_ENOMEM, "host allocation failed");
    int64_t *s_nb = stage.get();
    int32_t *s_src = (int32_t *)(s_nb + E), *s_dst = s_src + E, *s_flop = s_dst + E;
    if (E) {
        std::copy(edge_bytes, edge_bytes + E, s_nb);
        std::copy(edge_src, edge_src + E, s_src);
        std::copy(edge_dst, edge_dst + E, s_dst);
    }
    std::copy(flop, flop + K, s_flop);
    int64_t *d_nb = mem.as<int64_t>(), *d_out = d_nb + in64, *d_work = d_out + out64;
    const int32_t *d_src = (const int32_t *)(d_nb + E), *d_dst = d_src + E, *d_flop = d_dst + E;
    int32_t *d_first = (int32_t *)(d_out + 3);
    HIPCHK(hipMemcpyAsync(d_nb, stage.get(), in64 * 8, hipMemcpyHostToDevice, st));
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    HIPCHK(hipEventCreate(&ev0));
    HIPCHK(hipEventCreate(&ev1));
    struct EvGuard { hipEvent_t a, b; ~EvGuard() { (void)hipEventDestroy(a); (void)hipEventDestroy(b); } }
        guard{ev0, ev1};
    HIPCHK(hipEventRecord(ev0, st));
    HIPCHK(launch_cluster(st, d_flop, d_src, d_dst, d_nb, num_edges, K, L, cap, width,
                          cluster_work(d_work, K, L, width), d_out, d_first, nullptr, 0, exact, max_spins));
    HIPCHK(hipEventRecord(ev1, st));
    HIPCHK(hipMemcpyAsync(stage.get(), d_out, out64 * 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    const int64_t *res = stage.get();
    if (res[2] != 0) return fail(ALPA_DP_EHIP, "a wait between workgroups has run out");
    const int32_t *first = (const int32_t *)(res + 3);
    std::copy(first, first + L + 1, out_first_op);
    *out_comm = res[0];
    *out_sumsq = res[1];
    if (out_ms) HIPCHK(hipEventElapsedTime(out_ms, ev0, ev1));
    return ALPA_DP_OK;
}

extern "C" int alpa_cluster_layers(const int32_t *flop, int K, const int32_t *edge_src,
                                   const int32_t *edge_dst, const int64_t *edge_bytes,
                                   int num_edges, int L, int delta_ppm, int64_t *out_comm,
                                   int64_t *out_sumsq, int32_t *out_first_op, float *out_ms)
{
    return cluster_layers_impl(flop, K, edge_src, edge_dst, edge_bytes, num_edges, L, delta_ppm,
                               out_comm, out_sumsq, out_first_op, out_ms, 0);
}

extern "C" int alpa_cluster_layers_exact(const int32_t *flop, int K, const int32_t *edge_src,
                                         const int32_t *edge_dst, const int64_t *edge_bytes,
                                         int num_edges, int L, int delta_ppm, int64_t *out_comm,
                                         int64_t *out_sumsq, int32_t *out_first_op, float *out_ms)
{
    return cluster_layers_impl(flop, K, edge_src, edge_dst, edge_bytes, num_edges, L, delta_ppm,
                               out_comm, out_sumsq, out_first_op, out_ms, 1);
}

// alpa_cluster_layers with waits between workgroups of at most max_spins looks, for the test of a wait that runs out
// (not in the public header)
extern "C" int alpa_cluster_layers_waiting_(const int32_t *flop, int K, const int32_t *edge_src,
                                            const int32_t *edge_dst, const int64_t *edge_bytes,
                                            int num_edges, int L, int delta_ppm, int exact, unsigned max_spins,
                                            int64_t *out_comm, int64_t *out_sumsq, int32_t *out_first_op)
{
    return cluster_layers_impl(flop, K, edge_src, edge_dst, edge_bytes, num_edges, L, delta_ppm,
                               out_comm, out_sumsq, out_first_op, nullptr, exact, max_spins);
}

// ---------------------------------------------------------------- no allocation on the call

// Work memory of alpa_cluster_layers_static: what alpa_cluster_layers allocates per call, at
// the sizes of ALPA_CLUSTER_STATIC_MAX_OPS operators and layers with every operator feasible as
// first one, in int64 units (cluster_work_i64), and the two words of the argument checks.
namespace {
constexpr size_t SMAX = ALPA_CLUSTER_STATIC_MAX_OPS;
constexpr size_t SCRATCH_I64 = SMAX * SMAX + 2 * 129 * (SMAX + 1) + (SMAX + 1) + SMAX + 8 +
                               ((SMAX + 1) * (SMAX + 1) + 3) / 2 + 8;
}
// Every device the library runs on holds its own copy of this array until the process ends.  In
// host code the name is only a handle for hipGetSymbolAddress; kernels get the address below.
static __device__ __align__(256) int64_t scratch[SCRATCH_I64];

namespace {
constexpr int MAX_DEV = 64;
int64_t *g_scratch_of_device[MAX_DEV];      // device address of `scratch`, per device
bool g_scratch_known[MAX_DEV];
}

extern "C" int alpa_cluster_layers_static(const int32_t *d_flop, int K, const int32_t *d_edge_src,
                                          const int32_t *d_edge_dst, const int64_t *d_edge_bytes,
                                          int num_edges, int L, int delta_ppm, int64_t *d_out,
                                          int32_t *d_out_first_op, void *hip_stream)
{
    if (!d_flop || !d_out || !d_out_first_op) return fail(ALPA_DP_EINVAL, "null argument");
    if (K < 1 || L < 1) return fail(ALPA_DP_EINVAL, "K or L < 1");
    if (K > ALPA_CLUSTER_STATIC_MAX_OPS || L > ALPA_CLUSTER_STATIC_MAX_OPS)
        return fail(ALPA_DP_EINVAL, "K or L exceeds ALPA_CLUSTER_STATIC_MAX_OPS (the fixed work "
                                    "memory of this entry point); use alpa_cluster_layers");
    if (num_edges < 0 || (num_edges > 0 && (!d_edge_src || !d_edge_dst || !d_edge_bytes)))
        return fail(ALPA_DP_EINVAL, "edge list is null or num_edges < 0");
    if (delta_ppm < 0 || delta_ppm > 1000000000) return fail(ALPA_DP_EINVAL, "delta_ppm out of range");
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEV) return fail(ALPA_DP_EINVAL, "device index out of range");
    if (!g_scratch_known[dev]) {                   // set-up, once per device, that device current
        int64_t *ptr = nullptr;
        HIPCHK(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(ALPA_DP_EHIP, "hipGetSymbolAddress gave a null address");
        g_scratch_of_device[dev] = ptr;
        g_scratch_known[dev] = true;
    }
    int64_t *base = g_scratch_of_device[dev];
    if (cluster_work_i64(K, L, K) + 8 > SCRATCH_I64)
        return fail(ALPA_DP_EINVAL, "fixed work memory too small");        // (cannot be at the sizes above)
    int64_t *ctl = base;
    // Everything the kernels read from the work memory they have written in this call (cleared by
    // kernels, not a memset, so that the call can be recorded into a graph).
    HIPCHK(launch_cluster((hipStream_t)hip_stream, d_flop, d_edge_src, d_edge_dst, d_edge_bytes,
                          num_edges, K, L, /*cap=*/0, /*width=*/K, cluster_work(base + 8, K, L, K), d_out,
                          d_out_first_op, ctl, delta_ppm));
    return ALPA_DP_OK;
}
