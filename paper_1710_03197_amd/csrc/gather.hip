// Sample kernels that read the grid:
//   k_interp       V, a gather of J^d taps per sample (Section 2.1
//                  "Interpolation"), samples visited in grid-tile order.
//   k_grad         trajectory gradient through the derivative of the kernel.
// All arithmetic is float32 with float32 accumulation; window positions are
// float64 (u = omega * K/(2 pi) as one rounded multiply).
#include "device.h"

#include <type_traits>

namespace nufft {
namespace {

// ------------------------------------------------------------ V (gather)
// One workgroup per (bin, chunk), or per run of sparse tiles along the last
// axis: the tiles and their J-1 halo of the grid are staged in LDS once, then
// every sample of the item (window base inside the tiles) reads its J^d taps
// from LDS.
template <int J, int DIM>
__device__ __forceinline__ void interp_body(const InterpArgs &a, int64_t item, int gg) {
    extern __shared__ float2 reg[];
    const InterpItem it = a.items[item];
    int tc[DIM], base[DIM], E[DIM];
    {
        int t = it.bin;
#pragma unroll
        for (int ax = DIM - 1; ax >= 0; --ax) {
            tc[ax] = t % a.nt[ax];
            t /= a.nt[ax];
        }
    }
    // region: rows over the leading axes, each of P elements along the last
    // axis (its extent E made odd: the rows the lanes read then start in
    // different LDS banks)
    int rows = 1;
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
        base[ax] = tile_base(tc[ax], a.geo.K[ax], a.T[ax], a.nt[ax]);
        // a run of it.tiles tiles along the last axis, plus the J - 1 halo
        E[ax] = (ax == DIM - 1 ? it.tiles : 1) * a.T[ax] + J - 1;
        if (ax < DIM - 1) rows *= E[ax];
    }
    const int P = E[DIM - 1] | 1;
    const int region = rows * P;
    constexpr int TH = interp_threads(DIM);
    constexpr int SPT = kInterpSamplesPerThread;
    float w[SPT][DIM][J];
    int off[SPT];
    bool valid[SPT];
    float2 ph[SPT];
    int dst[SPT];  // caller's index of the sample (loaded early, used by the final store)
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
        const int s = threadIdx.x + k * TH;
        valid[k] = s < it.count;
        off[k] = 0;
        ph[k] = make_float2(1.f, 0.f);
        if (valid[k]) {
            const int64_t i = it.start + s;
            dst[k] = a.perm[i];
            int o = 0;
            if (a.geo.wtab) {
                // the window from the plan's table
                constexpr int NJ = table_taps_c(J);
                float4 r4[table_f4(DIM, NJ)];
                load_window_record<NJ, DIM>(a.geo, i, r4);
                int kw[DIM];
                float wt[DIM][NJ];
                unpack_window<NJ, DIM>(r4, kw, wt);
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) {
#pragma unroll
                    for (int j = 0; j < J; ++j) w[k][ax][j] = wt[ax][j];
                    o = o * (ax == DIM - 1 ? P : E[ax]) + (kw[ax] - base[ax]);
                }
            } else {
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) {
                    int kk[J];
                    const float f = window_pos<J>(a.geo, ax, a.om_sorted[i * DIM + ax], kk);
                    window_weights<J>(a.geo, a.geo.coef[ax], a.geo.nq[ax], f, w[k][ax]);
                    if (a.geo.minmax) mm_sign_taps<J>(w[k][ax], mm_wrap_from(a.geo, ax, a.om_sorted[i * DIM + ax]));
                    o = o * (ax == DIM - 1 ? P : E[ax]) + (kk[0] - base[ax]);
                }
            }
            off[k] = o;
            if (a.geo.minmax) ph[k] = mm_phase<DIM>(a.geo, a.om_sorted + i * DIM);
        }
    }
    // grid index of the first element of region row r (leading axes wrapped
    // at the grid's edge; the last axis is added by the caller)
    FastDiv byE1(DIM == 3 ? E[1] : 1);
    auto row_index = [&](int r) -> int64_t {
        if constexpr (DIM == 1) {
            return 0;
        } else if constexpr (DIM == 2) {
            int k0 = base[0] + r;
            if (k0 >= a.geo.K[0]) k0 -= a.geo.K[0];
            return int64_t(k0) * a.geo.K[1];
        } else {
            const int l0 = byE1.div(r);
            int k0 = base[0] + l0, k1 = base[1] + byE1.rem(r, l0);
            if (k0 >= a.geo.K[0]) k0 -= a.geo.K[0];
            if (k1 >= a.geo.K[1]) k1 -= a.geo.K[1];
            return (int64_t(k0) * a.geo.K[1] + k1) * a.geo.K[2];
        }
    };
    const int KL = a.geo.K[DIM - 1];
    const int H = (E[DIM - 1] + 1) >> 1;  // element pairs that cover a region row
    // pairs of the last axis in one 16-byte load: the grid's rows and the
    // region's first column must be even and the grid 16-byte aligned (a pair
    // then never straddles the wrap, K_last being even)
    const bool paired = (KL % 2 == 0) && (a.T[DIM - 1] % 2 == 0) && (a.grid_elems % 2 == 0) &&
                        (reinterpret_cast<uintptr_t>(a.G) % 16 == 0);
    // this thread's place in the row-major walk over the region's pairs: the
    // column stays fixed, the row advances by RP per round
    const int RP = H <= TH ? TH / H : 1;
    const int pr0 = H <= TH ? int(threadIdx.x) / H : 0;
    const int pc = H <= TH ? int(threadIdx.x) - pr0 * H : int(threadIdx.x);
    int kl = base[DIM - 1] + 2 * pc;  // grid column of the pair (< 2 K_last)
    if (kl >= KL) kl -= KL;
    const int g_lo = gg * a.grids_per_wg, g_hi = min(a.grids, g_lo + a.grids_per_wg);
    for (int g = g_lo; g < g_hi; ++g) {
        const float2 *G = a.G + int64_t(g) * a.grid_elems;
        __syncthreads();
        constexpr int U = 8;  // loads in flight per thread
        if (paired && H <= TH) {
            // (2D regions are a few rows: 2 paired loads keep the registers,
            // and the occupancy, of the element path)
            constexpr int UP = DIM == 3 ? U : 2;
            // rows of the region, H lanes per row, RP rows per round: the
            // NR rounds go in batches of up to U whose loads are issued
            // together (rows past the region clamped to its last row, so
            // every load is in bounds, and not stored); idle lanes
            // (pr0 >= RP) skip
            const float4 *G4 = reinterpret_cast<const float4 *>(G);
            auto rows_batch = [&](int u0, auto nu) {
                constexpr int NU = decltype(nu)::value;
                float4 v[NU];
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    v[u] = G4[(row_index(min(pr0 + (u0 + u) * RP, rows - 1)) + kl) >> 1];
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int r = pr0 + (u0 + u) * RP;
                    if (r < rows) {
                        float2 *dst = reg + r * P + 2 * pc;
                        dst[0] = make_float2(v[u].x, v[u].y);
                        if (2 * pc + 1 < P) dst[1] = make_float2(v[u].z, v[u].w);
                    }
                }
            };
            if (pr0 < RP) {
                const int NR = (rows + RP - 1) / RP;
                for (int u0 = 0; u0 < NR; u0 += UP) {
                    switch (min(UP, NR - u0)) {
                        case 1: rows_batch(u0, std::integral_constant<int, 1>()); break;
                        case 2: rows_batch(u0, std::integral_constant<int, 2>()); break;
                        case 3: rows_batch(u0, std::integral_constant<int, 3>()); break;
                        case 4: rows_batch(u0, std::integral_constant<int, 4>()); break;
                        case 5: rows_batch(u0, std::integral_constant<int, 5 <= UP ? 5 : 1>()); break;
                        case 6: rows_batch(u0, std::integral_constant<int, 6 <= UP ? 6 : 1>()); break;
                        case 7: rows_batch(u0, std::integral_constant<int, 7 <= UP ? 7 : 1>()); break;
                        default: rows_batch(u0, std::integral_constant<int, UP>()); break;
                    }
                }
            }
        } else {
            // element by element (odd tiles, unaligned grids, rows longer
            // than twice the workgroup), U elements per thread in flight
            FastDiv byP(P);
            for (int e0 = 0; e0 < region; e0 += U * TH) {
                float2 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = min(e0 + u * TH + int(threadIdx.x), region - 1);
                    const int r = byP.div(e);
                    int k = base[DIM - 1] + byP.rem(e, r);
                    if (k >= KL) k -= KL;
                    v[u] = G[row_index(r) + k];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * TH + threadIdx.x;
                    if (e < region) reg[e] = v[u];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            if (!valid[k]) continue;
            float2 acc = make_float2(0.f, 0.f);
            const float2 *r0 = reg + off[k];
            if constexpr (DIM == 1) {
#pragma unroll
                for (int j = 0; j < J; ++j) acc = cadd(acc, cscale(r0[j], w[k][0][j]));
            } else if constexpr (DIM == 2) {
#pragma unroll
                for (int j0 = 0; j0 < J; ++j0) {
                    const float2 *row = r0 + j0 * P;
                    float2 rs = make_float2(0.f, 0.f);
#pragma unroll
                    for (int j1 = 0; j1 < J; ++j1) rs = cadd(rs, cscale(row[j1], w[k][1][j1]));
                    acc = cadd(acc, cscale(rs, w[k][0][j0]));
                }
            } else {
                for (int j0 = 0; j0 < J; ++j0) {
                    float2 ps = make_float2(0.f, 0.f);
#pragma unroll
                    for (int j1 = 0; j1 < J; ++j1) {
                        const float2 *row = r0 + (j0 * E[1] + j1) * P;
                        float2 rs = make_float2(0.f, 0.f);
#pragma unroll
                        for (int j2 = 0; j2 < J; ++j2) rs = cadd(rs, cscale(row[j2], w[k][2][j2]));
                        ps = cadd(ps, cscale(rs, w[k][1][j1]));
                    }
                    acc = cadd(acc, cscale(ps, w[k][0][j0]));
                }
            }
            if (a.geo.minmax) acc = cmul(acc, ph[k]);
            a.y[int64_t(g) * a.M + dst[k]] = acc;
        }
    }
}

template <int J, int DIM>
__global__ __launch_bounds__(interp_threads(DIM)) void k_interp(InterpArgs a) {
    interp_body<J, DIM>(a, blockIdx.x, blockIdx.y);
}

template <int J, int DIM>
__global__ __launch_bounds__(interp_threads(DIM)) void k_interp_multi(const InterpArgs *__restrict__ jobs,
                                                     const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    interp_body<J, DIM>(jobs[b.x], b.y, b.z);
}

// Gather straight from the grid (L1/L2), one thread per sorted sample: used
// when the tile-plus-halo region does not fit the LDS budget.
template <int J, int DIM>
__device__ __forceinline__ void interp_direct_body(const InterpArgs &a, int64_t bx) {
    const int64_t i = bx * 256 + threadIdx.x;
    if (i >= a.M) return;
    float w[DIM][J];
    int kk[DIM][J];
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
        const float f = window_pos<J>(a.geo, ax, a.om_sorted[i * DIM + ax], kk[ax]);
        window_weights<J>(a.geo, a.geo.coef[ax], a.geo.nq[ax], f, w[ax]);
        if (a.geo.minmax) mm_sign_taps<J>(w[ax], mm_wrap_from(a.geo, ax, a.om_sorted[i * DIM + ax]));
    }
    const float2 ph = a.geo.minmax ? mm_phase<DIM>(a.geo, a.om_sorted + i * DIM) : make_float2(1.f, 0.f);
    const int64_t m = a.perm[i];
    for (int g = 0; g < a.grids; ++g) {
        const float2 *G = a.G + int64_t(g) * a.grid_elems;
        float2 acc = make_float2(0.f, 0.f);
        if constexpr (DIM == 1) {
#pragma unroll
            for (int j = 0; j < J; ++j) acc = cadd(acc, cscale(G[kk[0][j]], w[0][j]));
        } else if constexpr (DIM == 2) {
            const int64_t K1 = a.geo.K[1];
#pragma unroll
            for (int j0 = 0; j0 < J; ++j0) {
                const float2 *row = G + int64_t(kk[0][j0]) * K1;
                float2 rs = make_float2(0.f, 0.f);
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) rs = cadd(rs, cscale(row[kk[1][j1]], w[1][j1]));
                acc = cadd(acc, cscale(rs, w[0][j0]));
            }
        } else {
            const int64_t K1 = a.geo.K[1], K2 = a.geo.K[2];
            for (int j0 = 0; j0 < J; ++j0) {
                float2 ps = make_float2(0.f, 0.f);
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) {
                    const float2 *row = G + (int64_t(kk[0][j0]) * K1 + kk[1][j1]) * K2;
                    float2 rs = make_float2(0.f, 0.f);
#pragma unroll
                    for (int j2 = 0; j2 < J; ++j2) rs = cadd(rs, cscale(row[kk[2][j2]], w[2][j2]));
                    ps = cadd(ps, cscale(rs, w[1][j1]));
                }
                acc = cadd(acc, cscale(ps, w[0][j0]));
            }
        }
        if (a.geo.minmax) acc = cmul(acc, ph);
        a.y[int64_t(g) * a.M + m] = acc;
    }
}

template <int J, int DIM>
__global__ __launch_bounds__(256) void k_interp_direct(InterpArgs a) {
    interp_direct_body<J, DIM>(a, blockIdx.x);
}

template <int J, int DIM>
__global__ __launch_bounds__(256) void k_interp_direct_multi(const InterpArgs *__restrict__ jobs,
                                                            const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    interp_direct_body<J, DIM>(jobs[b.x], b.y);
}

// ------------------------------------------------------------ trajectory gradient
template <int J, int DIM>
__global__ __launch_bounds__(256) void k_grad(GradArgs a) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= a.M) return;
    float w[DIM][J], dw[DIM][J];
    int kk[DIM][J];
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
        const float f = window_pos<J>(a.geo, ax, a.om_sorted[i * DIM + ax], kk[ax]);
        window_weights<J>(a.geo, a.geo.coef[ax], a.geo.nq[ax], f, w[ax]);
        window_weights<J>(a.geo, a.geo.dcoef[ax], a.geo.nq_d[ax], f, dw[ax]);
    }
    const int64_t m = a.perm[i];
    float gsum[DIM];
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) gsum[ax] = 0.f;
    for (int g = 0; g < a.grids; ++g) {
        const float2 *G = a.G + int64_t(g) * a.grid_elems;
        float2 D[DIM];
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) D[ax] = make_float2(0.f, 0.f);
        if constexpr (DIM == 1) {
#pragma unroll
            for (int j = 0; j < J; ++j) D[0] = cadd(D[0], cscale(G[kk[0][j]], dw[0][j]));
        } else if constexpr (DIM == 2) {
            const int64_t K1 = a.geo.K[1];
#pragma unroll
            for (int j0 = 0; j0 < J; ++j0) {
                const float2 *row = G + int64_t(kk[0][j0]) * K1;
                float2 rs = make_float2(0.f, 0.f), rsd = make_float2(0.f, 0.f);
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) {
                    const float2 gv = row[kk[1][j1]];
                    rs = cadd(rs, cscale(gv, w[1][j1]));
                    rsd = cadd(rsd, cscale(gv, dw[1][j1]));
                }
                D[0] = cadd(D[0], cscale(rs, dw[0][j0]));
                D[1] = cadd(D[1], cscale(rsd, w[0][j0]));
            }
        } else {
            const int64_t K1 = a.geo.K[1], K2 = a.geo.K[2];
            for (int j0 = 0; j0 < J; ++j0) {
                float2 P = make_float2(0.f, 0.f), P1 = P, P2 = P;
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) {
                    const float2 *row = G + (int64_t(kk[0][j0]) * K1 + kk[1][j1]) * K2;
                    float2 rs = make_float2(0.f, 0.f), rsd = rs;
#pragma unroll
                    for (int j2 = 0; j2 < J; ++j2) {
                        const float2 gv = row[kk[2][j2]];
                        rs = cadd(rs, cscale(gv, w[2][j2]));
                        rsd = cadd(rsd, cscale(gv, dw[2][j2]));
                    }
                    P = cadd(P, cscale(rs, w[1][j1]));
                    P1 = cadd(P1, cscale(rs, dw[1][j1]));
                    P2 = cadd(P2, cscale(rsd, w[1][j1]));
                }
                D[0] = cadd(D[0], cscale(P, dw[0][j0]));
                D[1] = cadd(D[1], cscale(P1, w[0][j0]));
                D[2] = cadd(D[2], cscale(P2, w[0][j0]));
            }
        }
        const float2 gy = a.gy[int64_t(g) * a.M + m];
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) gsum[ax] += gy.x * D[ax].x + gy.y * D[ax].y;
    }
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) a.gom[m * DIM + ax] = gsum[ax] * float(a.geo.C[ax]);
}

// ------------------------------------------------------------ template dispatch
template <template <int, int> class Fn, int J>
struct DimDispatch {
    template <class... Args>
    static hipError_t run(int d, Args &&...args) {
        switch (d) {
            case 1: return Fn<J, 1>::go(args...);
            case 2: return Fn<J, 2>::go(args...);
            case 3: return Fn<J, 3>::go(args...);
            default: return hipErrorInvalidValue;
        }
    }
};

template <template <int, int> class Fn, class... Args>
hipError_t dispatch_jd(int J, int d, Args &&...args) {
    switch (J) {
#define NUFFT_J_CASE(JJ) \
    case JJ: return DimDispatch<Fn, JJ>::run(d, args...);
        NUFFT_J_CASE(2)
        NUFFT_J_CASE(3)
        NUFFT_J_CASE(4)
        NUFFT_J_CASE(5)
        NUFFT_J_CASE(6)
        NUFFT_J_CASE(7)
        NUFFT_J_CASE(8)
        NUFFT_J_CASE(9)
        NUFFT_J_CASE(10)
        NUFFT_J_CASE(11)
        NUFFT_J_CASE(12)
        NUFFT_J_CASE(13)
        NUFFT_J_CASE(14)
        NUFFT_J_CASE(15)
        NUFFT_J_CASE(16)
#undef NUFFT_J_CASE
        default: return hipErrorInvalidValue;
    }
}

template <int J, int DIM>
struct InterpLaunch {
    static hipError_t go(const InterpArgs &a, hipStream_t s) {
        if (a.M == 0) return hipSuccess;
        if (a.items) {
            if (a.n_items == 0) return hipSuccess;
            const unsigned gy = unsigned((a.grids + a.grids_per_wg - 1) / a.grids_per_wg);
            launch_kernel((k_interp<J, DIM>), dim3(unsigned(a.n_items), gy), dim3(interp_threads(DIM)), interp_lds(a), s, a);
        } else {
            const int64_t blocks = (a.M + 255) / 256;
            launch_kernel((k_interp_direct<J, DIM>), dim3(unsigned(blocks)), dim3(256), 0, s, a);
        }
        return hipGetLastError();
    }
};

template <int J, int DIM>
struct InterpMultiLaunch {
    static hipError_t go(const InterpArgs *jobs, const int4 *blocks, int64_t n, bool staged, size_t lds,
                         hipStream_t s) {
        if (n == 0) return hipSuccess;
        if (staged)
            launch_kernel((k_interp_multi<J, DIM>), dim3(unsigned(n)), dim3(interp_threads(DIM)), lds, s, jobs, blocks);
        else
            launch_kernel((k_interp_direct_multi<J, DIM>), dim3(unsigned(n)), dim3(256), 0, s, jobs, blocks);
        return hipGetLastError();
    }
};

template <int J, int DIM>
struct GradLaunch {
    static hipError_t go(const GradArgs &a, hipStream_t s) {
        if (a.M == 0) return hipSuccess;
        const int64_t blocks = (a.M + 255) / 256;
        launch_kernel((k_grad<J, DIM>), dim3(unsigned(blocks)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
};
}  // namespace

// ------------------------------------------------------------ launchers
size_t interp_lds(const InterpArgs &a) {
    if (!a.items) return 0;
    return size_t(interp_region_elems(a.geo.d, a.T, a.geo.J, a.merge)) * sizeof(float2);
}

hipError_t launch_interp(const InterpArgs &a, hipStream_t s) {
    return dispatch_jd<InterpLaunch>(a.geo.J, a.geo.d, a, s);
}

hipError_t launch_interp_multi(const InterpArgs *jobs, const int4 *blocks, int64_t nblocks, int J, int d,
                               bool staged, size_t lds, hipStream_t s) {
    return dispatch_jd<InterpMultiLaunch>(J, d, jobs, blocks, nblocks, staged, lds, s);
}

hipError_t launch_grad(const GradArgs &a, hipStream_t s) {
    return dispatch_jd<GradLaunch>(a.geo.J, a.geo.d, a, s);
}

}  // namespace nufft
