// Plan-time kernels (binning, the window table), sample permutation, density
// compensation and the L1TV image-domain steps.
#include "device.h"
#include <hipcub/hipcub.hpp>

#include <mutex>

namespace nufft {
namespace {

template <int NJ, int DIM>
__global__ __launch_bounds__(256) void k_weight_table(SampleGeom geo, const float *om_sorted, int64_t M, float *out) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= M) return;
    int kw[DIM];
    float w[DIM][NJ];
    eval_window<NJ, DIM>(geo, om_sorted + i * DIM, kw, w);
    float r[4 * table_f4(DIM, NJ)];
#pragma unroll
    for (int q = 0; q < 4 * table_f4(DIM, NJ); ++q) r[q] = 0.f;
    r[0] = __uint_as_float(unsigned(kw[0]) | (DIM > 1 ? unsigned(kw[1 < DIM ? 1 : 0]) << 16 : 0u));
    r[1] = __uint_as_float(DIM > 2 ? unsigned(kw[2 < DIM ? 2 : 0]) : 0u);
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) r[2 + ax * NJ + j] = w[ax][j];
    }
    float4 *dst = reinterpret_cast<float4 *>(out + i * (4 * table_f4(DIM, NJ)));
#pragma unroll
    for (int q = 0; q < table_f4(DIM, NJ); ++q) dst[q] = make_float4(r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
}

// ------------------------------------------------------------ plan-time binning
// key = (tile of the first tap) * 2^d + crossing code, bit a set when the
// window leaves the tile through its upper face along axis a.
__global__ __launch_bounds__(256) void k_bin_keys(BinArgs a) {
    const int64_t i0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t i = min(i0, a.M - 1);
    int key = 0, code = 0;
    bool bad = false;
    for (int ax = 0; ax < a.d; ++ax) {
        const float om = a.om[i * a.d + ax];
        int tile = 0;
        if (!isfinite(om)) {
            bad = true;
        } else {
            const double u = __dmul_rn(double(om), a.C[ax]);
            if (fabs(u) > 1.0e15) {
                bad = true;
            } else {
                const double k0 = floor(u - 0.5 * a.J) + 1.0;
                long long kw = static_cast<long long>(k0) % a.K[ax];
                if (kw < 0) kw += a.K[ax];
                tile = tile_of(int(kw), a.K[ax], a.T[ax], a.nt[ax]);
                if (a.nt[ax] > 1 && int(kw) + a.J - 1 >= tile_base(tile + 1, a.K[ax], a.T[ax], a.nt[ax]))
                    code |= 1 << ax;
            }
        }
        key = key * a.nt[ax] + tile;
    }
    key = (key << a.d) | code;
    if (bad) atomicOr(a.flag, 1);
    // Consecutive samples of a readout mostly share a sub-bin: one atomic per
    // run of equal keys in the wavefront (the crowded centre serialises them).
    // Lanes past the last sample end the last run.
    const bool live = i0 < a.M;
    const int lane = threadIdx.x & 63;
    const int before = __shfl_up(key, 1);
    const uint64_t heads = __ballot(!live || lane == 0 || key != before);
    if (!live) return;
    a.keys[i] = key;
    if ((heads >> lane) & 1u) {
        const uint64_t rest = lane == 63 ? 0 : heads >> (lane + 1);
        atomicAdd(&a.counts[key], rest ? int(__builtin_ctzll(rest)) + 1 : 64 - lane);
    }
}

__global__ void k_iota(int *v, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) v[i] = int(i);
}

__device__ __forceinline__ void permute_samples_body(const float2 *y, const int *perm, int64_t M, int grids,
                                                     float2 *ys, int64_t bx) {
    const int64_t i = bx * 256 + threadIdx.x;
    if (i >= M) return;
    const int64_t m = perm[i];
    for (int g = 0; g < grids; ++g) ys[int64_t(g) * M + i] = y[int64_t(g) * M + m];
}

__global__ __launch_bounds__(256) void k_permute_samples(const float2 *y, const int *perm, int64_t M, int grids,
                                                         float2 *ys) {
    permute_samples_body(y, perm, M, grids, ys, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_permute_samples_multi(const PermuteJob *__restrict__ jobs,
                                                               const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const PermuteJob &j = jobs[b.x];
    permute_samples_body(j.y, j.perm, j.M, j.grids, j.ys, b.y);
}

__global__ void k_permute_points(const float *om, const int *perm, int64_t M, int d, float *out) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int64_t m = perm[i];
    for (int ax = 0; ax < d; ++ax) out[i * d + ax] = om[m * d + ax];
}

// ------------------------------------------------------------ density compensation
// One fixed-point step of the sampling-density weights (Pipe-Menon) with the
// kernel normalised to peak 1: the gridding ran on wc = w * inv_c and
// u = V V^H wc with the unnormalised kernel (peak c = prod_a I0(beta_a)), so
// |u| * inv_c is the normalised V V^H w;  w[m] <- w[m] / (|u[m]| * inv_c)
// (a zero or non-finite quotient keeps w[m]), and wc is refreshed for the
// next gridding.  The 1/c pre-scaling keeps the grid values near the
// weights' own scale (c^2d overflows float32 for d = 3 and J >= 8).  u and wc
// are in the plan's sorted order, which the gridding reads and the gather
// writes without a permutation; only the weights go through it.
__global__ __launch_bounds__(256) void k_dc_update(float *w, const int *perm, const float2 *u, float2 *wc, int64_t M,
                                                   float inv_c) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int m = perm[i];
    const float a = hypotf(u[i].x, u[i].y) * inv_c;
    float v = w[m];
    if (a > 0.f && isfinite(a)) v = v / a;
    w[m] = v;
    wc[i] = make_float2(v * inv_c, 0.f);
}

__global__ __launch_bounds__(256) void k_weights_to_samples(const float *w, const int *perm, float2 *wc, int64_t M,
                                                            float scale) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < M) wc[i] = make_float2(w[perm[i]] * scale, 0.f);
}

// ------------------------------------------------------------ TV split-Bregman pieces
// Image gradient grad_a x = x(.., i_a + 1, ..) - x(.., i_a, ..) with
// wrap-around, its transpose g(.., i_a - 1, ..) - g(.., i_a, ..), and the
// complex soft threshold shrink(z, t) = z / |z| * max(|z| - t, 0).  One
// thread per pixel; every axis of the pixel in registers.
struct TvGeom {
    int d;
    int64_t N[kMaxDim];
    int64_t stride[kMaxDim];
    int64_t n;
};

__device__ __forceinline__ float2 shrinkc(float2 z, float t) {
    const float a = hypotf(z.x, z.y);
    const float sc = a > t ? (a - t) / a : 0.f;
    return make_float2(z.x * sc, z.y * sc);
}

// index of the pixel one step along axis a (delta = +1 or -1), wrapped
__device__ __forceinline__ int64_t tv_step(const TvGeom &g, int64_t i, int a, int delta) {
    const int64_t c = (i / g.stride[a]) % g.N[a];
    int64_t c2 = c + delta;
    if (c2 < 0) c2 += g.N[a];
    if (c2 >= g.N[a]) c2 -= g.N[a];
    return i + (c2 - c) * g.stride[a];
}

__global__ __launch_bounds__(256) void k_tv_shrink(TvGeom g, const float2 *x, float2 *dd, float2 *bb, float t) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const float2 xi = x[i];
    for (int a = 0; a < g.d; ++a) {
        const float2 xn = x[tv_step(g, i, a, +1)];
        const int64_t k = int64_t(a) * g.n + i;
        const float2 z = cadd(csub(xn, xi), bb[k]);
        const float2 dv = shrinkc(z, t);
        dd[k] = dv;
        bb[k] = csub(z, dv);
    }
}

__global__ __launch_bounds__(256) void k_tv_rhs(TvGeom g, float mu, const float2 *ahy, const float2 *df,
                                                const float2 *bf, float lam, const float2 *dd, const float2 *bb,
                                                float2 *rhs) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    float2 v = ahy[i];
    if (df) v = cadd(v, csub(df[i], bf[i]));
    float2 acc = cscale(v, mu);
    for (int a = 0; a < g.d; ++a) {
        const int64_t k = int64_t(a) * g.n;
        const int64_t ip = tv_step(g, i, a, -1);
        const float2 here = csub(dd[k + i], bb[k + i]);
        const float2 prev = csub(dd[k + ip], bb[k + ip]);
        acc = cadd(acc, cscale(csub(prev, here), lam));
    }
    rhs[i] = acc;
}

__global__ __launch_bounds__(256) void k_tv_normal(TvGeom g, float mu, const float2 *ahax, float lam, const float2 *x,
                                                   float2 *out) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const float2 xi = x[i];
    float2 lap = make_float2(0.f, 0.f);
    for (int a = 0; a < g.d; ++a) {
        // grad^T grad along a: 2 x(i) - x(i - e_a) - x(i + e_a)
        const float2 xm = x[tv_step(g, i, a, -1)];
        const float2 xp = x[tv_step(g, i, a, +1)];
        lap = cadd(lap, csub(csub(cscale(xi, 2.f), xm), xp));
    }
    out[i] = cadd(cscale(ahax[i], mu), cscale(lap, lam));
}

__global__ __launch_bounds__(256) void k_bregman_shrink(int64_t n, const float2 *r, float2 *dv, float2 *bv, float t) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float2 z = cadd(r[i], bv[i]);
    const float2 dd = shrinkc(z, t);
    dv[i] = dd;
    bv[i] = csub(z, dd);
}

}  // namespace

// ------------------------------------------------------------ launchers
hipError_t launch_permute_samples_multi(const PermuteJob *jobs, const int4 *blocks, int64_t nblocks, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    launch_kernel(k_permute_samples_multi, dim3(unsigned(nblocks)), dim3(256), 0, s, jobs, blocks);
    return hipGetLastError();
}

hipError_t launch_bin_keys(const BinArgs &a, hipStream_t s) {
    if (a.M == 0) return hipSuccess;
    const int64_t blocks = (a.M + 255) / 256;
    launch_kernel(k_bin_keys, dim3(unsigned(blocks)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dc_update(float *w, const int *perm, const float2 *u, float2 *wc, int64_t M, float inv_c, hipStream_t s) {
    if (M == 0) return hipSuccess;
    launch_kernel(k_dc_update, dim3(unsigned((M + 255) / 256)), dim3(256), 0, s, w, perm, u, wc, M, inv_c);
    return hipGetLastError();
}

template <int NJ>
hipError_t launch_weight_table_j(const SampleGeom &g, const float *om_sorted, int64_t M, float *out, hipStream_t s) {
    const dim3 grid(unsigned((M + 255) / 256));
    switch (g.d) {
        case 1: launch_kernel((k_weight_table<NJ, 1>), grid, dim3(256), 0, s, g, om_sorted, M, out); break;
        case 2: launch_kernel((k_weight_table<NJ, 2>), grid, dim3(256), 0, s, g, om_sorted, M, out); break;
        case 3: launch_kernel((k_weight_table<NJ, 3>), grid, dim3(256), 0, s, g, om_sorted, M, out); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_weight_table(const SampleGeom &g, const float *om_sorted, int64_t M, float *out, hipStream_t s) {
    if (M == 0) return hipSuccess;
    if (g.wtab_stride != table_stride(g.d, g.J)) return hipErrorInvalidValue;
    switch (table_taps(g.J)) {
        case 6: return launch_weight_table_j<6>(g, om_sorted, M, out, s);
        case 8: return launch_weight_table_j<8>(g, om_sorted, M, out, s);
        default: return launch_weight_table_j<16>(g, om_sorted, M, out, s);
    }
}

hipError_t launch_weights_to_samples(const float *w, const int *perm, float2 *wc, int64_t M, float scale,
                                     hipStream_t s) {
    if (M == 0) return hipSuccess;
    launch_kernel(k_weights_to_samples, dim3(unsigned((M + 255) / 256)), dim3(256), 0, s, w, perm, wc, M, scale);
    return hipGetLastError();
}

// ---- fixed device scratch of the allocation-free density compensation
// The two complex sample buffers of the iteration (the weights handed to the
// gridding, and V V^H of them), kDcScratchMaxM samples each, as one static
// device array: every GPU the library runs on holds its own copy from the
// first use until the process ends.  Host code never passes the array's name
// to a kernel (on the host it is only a stand-in for the symbol); it uses the
// device address that hipGetSymbolAddress returns, looked up once per device
// with that device current.
static __device__ __align__(256) float2 scratch[2 * kDcScratchMaxM];

hipError_t dc_scratch(float2 **wc, float2 **u) {
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *wc = static_cast<float2 *>(addr[dev]);
    *u = *wc + kDcScratchMaxM;
    return hipSuccess;
}

static TvGeom tv_geom(int d, const int64_t *N) {
    TvGeom g{};
    g.d = d;
    int64_t st = 1;
    for (int a = d - 1; a >= 0; --a) {
        g.N[a] = N[a];
        g.stride[a] = st;
        st *= N[a];
    }
    g.n = st;
    return g;
}

hipError_t launch_tv_shrink(int d, const int64_t *N, const float2 *x, float2 *dd, float2 *bb, float t, hipStream_t s) {
    const TvGeom g = tv_geom(d, N);
    if (g.n == 0) return hipSuccess;
    launch_kernel(k_tv_shrink, dim3(unsigned((g.n + 255) / 256)), dim3(256), 0, s, g, x, dd, bb, t);
    return hipGetLastError();
}

hipError_t launch_tv_rhs(int d, const int64_t *N, float mu, const float2 *ahy, const float2 *df, const float2 *bf,
                         float lam, const float2 *dd, const float2 *bb, float2 *rhs, hipStream_t s) {
    const TvGeom g = tv_geom(d, N);
    if (g.n == 0) return hipSuccess;
    launch_kernel(k_tv_rhs, dim3(unsigned((g.n + 255) / 256)), dim3(256), 0, s, g, mu, ahy, df, bf, lam, dd, bb,
                       rhs);
    return hipGetLastError();
}

hipError_t launch_tv_normal(int d, const int64_t *N, float mu, const float2 *ahax, float lam, const float2 *x,
                            float2 *out, hipStream_t s) {
    const TvGeom g = tv_geom(d, N);
    if (g.n == 0) return hipSuccess;
    launch_kernel(k_tv_normal, dim3(unsigned((g.n + 255) / 256)), dim3(256), 0, s, g, mu, ahax, lam, x, out);
    return hipGetLastError();
}

hipError_t launch_bregman_shrink(int64_t n, const float2 *r, float2 *dv, float2 *bv, float t, hipStream_t s) {
    if (n == 0) return hipSuccess;
    launch_kernel(k_bregman_shrink, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, r, dv, bv, t);
    return hipGetLastError();
}

hipError_t launch_iota(int *v, int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    launch_kernel(k_iota, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, v, n);
    return hipGetLastError();
}

hipError_t launch_permute_samples(const float2 *y, const int *perm, int64_t M, int grids, float2 *ys,
                                  hipStream_t s) {
    if (M == 0 || grids == 0) return hipSuccess;
    launch_kernel(k_permute_samples, dim3(unsigned((M + 255) / 256)), dim3(256), 0, s, y, perm, M, grids, ys);
    return hipGetLastError();
}

hipError_t launch_permute_points(const float *om, const int *perm, int64_t M, int d, float *om_sorted,
                                 hipStream_t s) {
    if (M == 0) return hipSuccess;
    launch_kernel(k_permute_points, dim3(unsigned((M + 255) / 256)), dim3(256), 0, s, om, perm, M, d,
                       om_sorted);
    return hipGetLastError();
}

hipError_t sort_pairs_temp_bytes(int64_t n, int key_bits, size_t *bytes) {
    *bytes = 0;
    if (n == 0) return hipSuccess;
    return hipcub::DeviceRadixSort::SortPairs(nullptr, *bytes, static_cast<const int *>(nullptr),
                                              static_cast<int *>(nullptr), static_cast<const int *>(nullptr),
                                              static_cast<int *>(nullptr), int(n), 0, key_bits);
}

hipError_t sort_pairs(const int *keys_in, int *keys_out, const int *vals_in, int *vals_out, int64_t n,
                      int key_bits, void *temp, size_t temp_bytes, hipStream_t s) {
    if (n == 0) return hipSuccess;
    size_t need = 0;
    hipError_t e = sort_pairs_temp_bytes(n, key_bits, &need);
    if (e != hipSuccess) return e;
    if (need > temp_bytes || !temp) return hipErrorInvalidValue;
    return hipcub::DeviceRadixSort::SortPairs(temp, temp_bytes, keys_in, keys_out, vals_in, vals_out, int(n), 0,
                                              key_bits, s);
}

}  // namespace nufft
