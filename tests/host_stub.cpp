// HIP runtime and kernel launchers for host-only tests of the runtime: "device"
// memory is host memory, launches are written to a log instead of run.  Linked
// with api.cpp and kb_host.cpp into a library without any device code, so a
// test can see on the CPU which streams a call waits for, what it allocates
// and what it would launch, and can make an allocation fail.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

#include "nufft_internal.h"

namespace {
std::string g_log;
std::map<const char *, size_t> g_live;  // allocations
size_t g_fail_from = SIZE_MAX;          // allocations of at least this many bytes fail ...
int g_fail_count = 0;                   // ... this many times

void note(const char *fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_log += buf;
    g_log += '\n';
}

bool live(const void *p) {
    auto it = g_live.upper_bound(static_cast<const char *>(p));
    if (it == g_live.begin()) return false;
    --it;
    return static_cast<const char *>(p) < it->first + it->second;
}
}  // namespace

extern "C" {
const char *stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_fail_allocations(size_t from_bytes, int count) {
    g_fail_from = from_bytes;
    g_fail_count = count;
}
size_t stub_live_bytes() {
    size_t n = 0;
    for (auto &a : g_live) n += a.second;
    return n;
}

hipError_t hipMalloc(void **p, size_t bytes) {
    if (bytes >= g_fail_from && g_fail_count > 0) {
        --g_fail_count;
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    // address space only: a test may hold grids larger than the host's memory
    void *m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    g_live[static_cast<const char *>(m)] = bytes;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = g_live.find(static_cast<const char *>(p));
    if (it == g_live.end()) return hipErrorInvalidValue;
    munmap(p, it->second);
    g_live.erase(it);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    if (kind != hipMemcpyDeviceToHost) note("write stream=%p", static_cast<void *>(st));
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    note("sync stream=%p", static_cast<void *>(s));
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = nullptr, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    return *x = nullptr, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}  // extern "C"

namespace nufft {

// Samples with a negative first coordinate all fall into the first sub-bin,
// the others are dealt over all sub-bins.
hipError_t launch_bin_keys(const BinArgs &a, hipStream_t) {
    int64_t nkeys = 1;
    for (int ax = 0; ax < a.d; ++ax) nkeys *= a.nt[ax];
    nkeys <<= a.d;
    for (int64_t i = 0; i < a.M; ++i) {
        if (!std::isfinite(a.om[i * a.d])) *a.flag = 1;
        ++a.counts[a.om[i * a.d] < 0.f ? 0 : i % nkeys];
    }
    return hipSuccess;
}
hipError_t launch_iota(int *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t sort_pairs_temp_bytes(int64_t, int, size_t *bytes) { return *bytes = 1, hipSuccess; }
hipError_t sort_pairs(const int *, int *, const int *, int *, int64_t, int, void *, size_t, hipStream_t s) {
    note("write stream=%p", static_cast<void *>(s));
    return hipSuccess;
}
hipError_t launch_permute_points(const float *, const int *, int64_t, int, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_weight_table(const SampleGeom &, const float *, int64_t, float *, hipStream_t) {
    note("table");
    return hipSuccess;
}

FftLaunch first_pass_launch(const FirstPassArgs &, int) { return {64, 1, 0, 1, 1}; }
FftLaunch strided_pass_launch(const StridedPassArgs &, int) { return {64, 1, 0, 1, 1}; }
FftLaunch last_pass_launch(const LastPassArgs &, int) { return {64, 1, 0, 1, 1}; }
hipError_t launch_strided_pass(const StridedPassArgs &a, hipStream_t) {
    note("strided inverse=%d wide=%d", a.inverse, strided_wide(a));
    return hipSuccess;
}
hipError_t launch_strided_pass_multi(const StridedJob *jobs, const int4 *, int64_t, int, bool inverse, bool, bool wide,
                                     size_t, hipStream_t) {
    note("strided_multi K=%d inverse=%d wide=%d", jobs[0].a.K, inverse, wide);
    return hipSuccess;
}
hipError_t launch_first_pass(const FirstPassArgs &a, hipStream_t) {
    float s = 1.0f;  // the first pixel's scale, multiplied as the kernel does
    for (int ax = a.d - 2; ax >= 0; --ax) s *= a.scale[ax][0];
    note("first K=%d scale=%a", a.K, a.scale[a.d - 1][0] * s);
    return hipSuccess;
}
hipError_t launch_last_pass(const LastPassArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_first_pass_multi(const FirstJob *, const int4 *, int64_t, int, bool, size_t, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_last_pass_multi(const LastJob *, const int4 *, int64_t, int, bool, size_t, hipStream_t) {
    return hipSuccess;
}

int grid_variant(const GridArgs &a) { return a.cols; }
size_t grid_lds(const GridArgs &) { return 0; }
size_t interp_lds(const InterpArgs &) { return 0; }
int grid_groups(const GridArgs &a) {
    const int gp = a.cols ? kColGrids : a.mfma ? a.grids_per_wg : 1;
    return (a.grids + gp - 1) / gp;
}
hipError_t launch_grid(const GridArgs &a, hipStream_t) {
    const bool ok = live(a.items) && live(a.item_segs) && live(a.h) && (!a.geo.wtab || live(a.geo.wtab));
    note("grid items=%lld cols=%d table=%d live=%d", static_cast<long long>(a.n_items), a.cols, a.geo.wtab != nullptr,
         ok || a.n_items == 0);
    return hipSuccess;
}
hipError_t launch_interp(const InterpArgs &a, hipStream_t) {
    const bool ok = live(a.items) && live(a.G) && (!a.geo.wtab || live(a.geo.wtab));
    note("interp items=%lld grids_per_wg=%d table=%d live=%d", static_cast<long long>(a.n_items), a.grids_per_wg,
         a.geo.wtab != nullptr, ok || a.n_items == 0);
    return hipSuccess;
}
hipError_t launch_grid_multi(const GridArgs *, const int4 *, int64_t blocks, const GridArgs &proto, size_t,
                             hipStream_t) {
    note("grid_multi blocks=%lld cols=%d", static_cast<long long>(blocks), proto.cols);
    return hipSuccess;
}
hipError_t launch_interp_multi(const InterpArgs *jobs, const int4 *, int64_t blocks, int, int, bool, size_t,
                               hipStream_t) {
    note("interp_multi blocks=%lld grids_per_wg=%d", static_cast<long long>(blocks), jobs[0].grids_per_wg);
    return hipSuccess;
}
hipError_t launch_reduce_partials(const ReduceArgs &a, hipStream_t) {
    note("reduce live=%d", live(a.hot) && live(a.partials));
    return hipSuccess;
}
hipError_t launch_reduce_partials_multi(const ReduceArgs *, const int4 *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_permute_samples(const float2 *, const int *, int64_t, int, float2 *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_permute_samples_multi(const PermuteJob *, const int4 *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_grad(const GradArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_dc_update(float *, const int *, const float2 *, float2 *, int64_t, float, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_weights_to_samples(const float *, const int *, float2 *, int64_t, float, hipStream_t) {
    return hipSuccess;
}
hipError_t dc_scratch(float2 **, float2 **) { return hipErrorInvalidValue; }
hipError_t launch_tv_shrink(int, const int64_t *, const float2 *, float2 *, float2 *, float, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_tv_rhs(int, const int64_t *, float, const float2 *, const float2 *, const float2 *, float,
                         const float2 *, const float2 *, float2 *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_tv_normal(int, const int64_t *, float, const float2 *, float, const float2 *, float2 *,
                            hipStream_t) {
    return hipSuccess;
}
hipError_t launch_bregman_shrink(int64_t, const float2 *, float2 *, float2 *, float, hipStream_t) {
    return hipSuccess;
}

}  // namespace nufft
