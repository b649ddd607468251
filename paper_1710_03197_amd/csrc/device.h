// Device helpers shared by the kernel sources: launches, complex arithmetic,
// division by launch constants, and the interpolation window of a sample.
#pragma once

#include <hip/hip_ext.h>

#include <algorithm>

#include "nufft_internal.h"

namespace nufft {
namespace {

// Every kernel launch of the library: a launch inside a timed stage carries the
// stage's start and stop events.
template <typename K, typename... Args>
void launch_kernel(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, Args... args) {
    LaunchEvents *ev = g_launch_events;
    if (ev && !ev->used) {
        ev->used = true;
        hipExtLaunchKernelGGL(kernel, grid, block, uint32_t(lds), s, ev->start, ev->stop, 0u, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
    }
}

// ------------------------------------------------------------ complex helpers
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__device__ __forceinline__ float2 cmulcj(float2 a, float2 b) {
    return make_float2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 mul_negi(float2 a) { return make_float2(a.y, -a.x); }

// floor(e / D) for a divisor D >= 1 fixed per launch: q = floor(e m / 2^32)
// with m = ceil(2^32 / D) is exact whenever e (D - 1) < 2^32, since the error
// e (m D - 2^32) / (D 2^32) then stays below 1/D.  One high multiply instead
// of an integer division.  Every use here divides tile positions (< 4096) by
// at most 4096, or a column index c < K_1 K_2 by K_2 with K_1 K_2^2 < 2^32
// (checked when the plan is made).
struct FastDiv {
    unsigned m;
    int d;
    __device__ __forceinline__ FastDiv() : m(0u), d(1) {}
    __device__ __forceinline__ explicit FastDiv(int D)  // D uniform: one scalar register
        : m(__builtin_amdgcn_readfirstlane(D > 1 ? 0xFFFFFFFFu / unsigned(D) + 1u : 0u)), d(D) {}
    __device__ __forceinline__ FastDiv(unsigned magic, int D) : m(magic), d(D) {}  // magic made on the host
    __device__ __forceinline__ int div(int e) const { return d > 1 ? int(__umulhi(unsigned(e), m)) : e; }
    __device__ __forceinline__ int rem(int e, int q) const { return e - __umul24(q, d); }
};

// ------------------------------------------------------------ interpolation window
// k0 mod K for an integer-valued k0 (|k0| <= 1e15, checked when the plan is
// made).  Trajectories inside [-pi, pi) give |k0| <= K/2 + J/2 < K, handled
// without the 64-bit division the general case needs.
__device__ __forceinline__ int wrap_first_tap(double k0, int K) {
    const double Kd = double(K);
    if (k0 >= 0.0 && k0 < Kd) return int(k0);
    if (k0 < 0.0 && k0 >= -Kd) return int(k0) + K;
    long long kw = static_cast<long long>(k0) % K;
    if (kw < 0) kw += K;
    return int(kw);
}


// First tap k0 = floor(u - J/2) + 1 with u = omega * K/(2 pi) in float64, the
// J wrapped grid indices and the offset f = u - k0 - (J/2 - 1) in [0, 1).
template <int J>
__device__ __forceinline__ float window_pos(const SampleGeom &geo, int ax, float om, int *kk) {
    const double u = __dmul_rn(double(om), geo.C[ax]);
    const double k0 = floor(u - 0.5 * J) + 1.0;
    const float f = float(u - k0 - (0.5 * J - 1.0));
    const int K = geo.K[ax];
    const int kw = wrap_first_tap(k0, K);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        int k = kw + j;
        kk[j] = k >= K ? k - K : k;
    }
    return f;
}

// Min-max interpolator: the coefficients are c_j = e^{i gamma t_j / 2} c'_j
// with c' the real fitted factors, and e^{i gamma t_j / 2} =
// e^{i omega / 2} (-1)^{floor(k0 / K)} (-1)^{[k0 mod K + j >= K]} e^{-i pi k_w / K}
// (k_w the wrapped grid index).  The FFT passes apply e^{-i pi k_w / K}; the
// sample kernels apply the rest: this per-sample phase (float64 angle) and a
// sign on taps that wrap past K.
template <int DIM>
__device__ __forceinline__ float2 mm_phase(const SampleGeom &geo, const float *om) {
    double ang = 0.0;
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
        const double u = __dmul_rn(double(om[ax]), geo.C[ax]);
        const double k0 = floor(u - 0.5 * geo.J) + 1.0;
        ang += 0.5 * double(om[ax]) + 3.141592653589793 * floor(k0 / double(geo.K[ax]));
    }
    double sn, cs;
    sincos(ang, &sn, &cs);
    return make_float2(float(cs), float(sn));
}

// First tap index j that wraps past K on axis `ax` (J or more: none).
__device__ __forceinline__ int mm_wrap_from(const SampleGeom &geo, int ax, float om) {
    const double u = __dmul_rn(double(om), geo.C[ax]);
    const double k0 = floor(u - 0.5 * geo.J) + 1.0;
    const int K = geo.K[ax];
    return K - wrap_first_tap(k0, K);
}

template <int NJ>
__device__ __forceinline__ void mm_sign_taps(float *w, int wrap_from) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        if (j >= wrap_from) w[j] = -w[j];
}

// Per-tap polynomials of the kernel fit: NJ Horner chains in z over the
// coefficient rows (highest degree first, zero padded to a multiple of 2
// rows).  The table is the same for every lane, so it is read through the
// constant address space, which the compiler serves with scalar loads; a row
// pair is fetched at once instead of one dependent load per step.
typedef const __attribute__((address_space(4))) float const_float;

template <int NJ>
__device__ __forceinline__ void poly_rows(const float *rows, int jp, int nq, float z, float *w) {
    const_float *r = (const_float *)rows;
    float v[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) v[j] = 0.f;
    for (int q = 0; q < nq; q += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) v[j] = fmaf(v[j], z, r[(q + u) * jp + j]);
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = v[j];
}

// w_j(f), j < J: the kernel weights of the window whose first tap is at
// fractional offset f.
template <int J>
__device__ __forceinline__ void window_weights(const SampleGeom &geo, const float *rows, int nq, float f, float *w) {
    poly_rows<J>(rows, geo.jp, nq, 2.0f * f - 1.0f, w);
}

// ---- the plan's window table (optional): one record per sorted sample
constexpr int table_taps_c(int J) { return J <= 6 ? 6 : J <= 8 ? 8 : 16; }
constexpr int table_f4(int DIM, int NJ) { return (2 + DIM * NJ + 3) / 4; }

// Window of sorted sample i on every axis: wrapped first taps and the NJ
// weights (zero past J), evaluated exactly as the table records them.
template <int NJ, int DIM>
__device__ __forceinline__ void eval_window(const SampleGeom &geo, const float *om, int *kw, float (*w)[NJ]) {
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
        const double u = __dmul_rn(double(om[ax]), geo.C[ax]);
        const double k0 = floor(u - 0.5 * geo.J) + 1.0;
        const float f = float(u - k0 - (0.5 * geo.J - 1.0));
        kw[ax] = wrap_first_tap(k0, geo.K[ax]);
        poly_rows<NJ>(geo.coef[ax], geo.jp, geo.nq[ax], 2.0f * f - 1.0f, w[ax]);
    }
}

// Unpacks a record already loaded as float4s.
template <int NJ, int DIM>
__device__ __forceinline__ void unpack_window(const float4 *r4, int *kw, float (*w)[NJ]) {
    float r[4 * table_f4(DIM, NJ)];
#pragma unroll
    for (int q = 0; q < table_f4(DIM, NJ); ++q) {
        r[4 * q] = r4[q].x;
        r[4 * q + 1] = r4[q].y;
        r[4 * q + 2] = r4[q].z;
        r[4 * q + 3] = r4[q].w;
    }
    const unsigned k01 = __float_as_uint(r[0]), k2 = __float_as_uint(r[1]);
    kw[0] = int(k01 & 0xffffu);
    if (DIM > 1) kw[1 < DIM ? 1 : 0] = int(k01 >> 16);
    if (DIM > 2) kw[2 < DIM ? 2 : 0] = int(k2 & 0xffffu);
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) w[ax][j] = r[2 + ax * NJ + j];
    }
}

template <int NJ, int DIM>
__device__ __forceinline__ void load_window_record(const SampleGeom &geo, int64_t i, float4 *r4) {
    const float4 *src = reinterpret_cast<const float4 *>(geo.wtab + i * geo.wtab_stride);
#pragma unroll
    for (int q = 0; q < table_f4(DIM, NJ); ++q) r4[q] = src[q];
}

}  // namespace
}  // namespace nufft
