// FFT kernels of the pair (paper Section 2.1 "Oversampled FFT"):
//   k_first_pass   S + zero padding + FFT along the contiguous last axis
//                  (Section 2.1 "Scaling", "Oversampled FFT"); the pad is index
//                  arithmetic on the load, never a materialised array.
//   k_strided_pass FFT along a strided axis, zero-padded input rows (forward) or
//                  cropped output rows (adjoint, the copy after the IFFT).
//   k_last_pass    inverse FFT along the last axis + crop + S^H + coil combine
//                  (Section 2.2, multi-coil: sum_i conj(c_i) A^H y_i).
// All arithmetic is float32.
#include <type_traits>

#include "device.h"

namespace nufft {
namespace {

// ------------------------------------------------------------ small DFTs (e^{-2 pi i / R})
template <int R>
__device__ __forceinline__ void dft(float2 *v);

template <>
__device__ __forceinline__ void dft<2>(float2 *v) {
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <>
__device__ __forceinline__ void dft<3>(float2 *v) {
    const float c = 0.86602540378443864676f;  // sin(2 pi / 3)
    float2 s = cadd(v[1], v[2]), dd = csub(v[1], v[2]);
    float2 m = make_float2(v[0].x - 0.5f * s.x, v[0].y - 0.5f * s.y);
    v[0] = cadd(v[0], s);
    v[1] = make_float2(m.x + c * dd.y, m.y - c * dd.x);
    v[2] = make_float2(m.x - c * dd.y, m.y + c * dd.x);
}

template <>
__device__ __forceinline__ void dft<4>(float2 *v) {
    float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    float2 t2 = cadd(v[1], v[3]), t3 = mul_negi(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
}

template <>
__device__ __forceinline__ void dft<5>(float2 *v) {
    const float c1 = 0.30901699437494742410f, c2 = -0.80901699437494742410f;
    const float s1 = 0.95105651629515357212f, s2 = 0.58778525229247312917f;
    float2 p1 = cadd(v[1], v[4]), m1 = csub(v[1], v[4]);
    float2 p2 = cadd(v[2], v[3]), m2 = csub(v[2], v[3]);
    float2 x0 = v[0];
    float2 A1 = make_float2(x0.x + c1 * p1.x + c2 * p2.x, x0.y + c1 * p1.y + c2 * p2.y);
    float2 B1 = make_float2(s1 * m1.x + s2 * m2.x, s1 * m1.y + s2 * m2.y);
    float2 A2 = make_float2(x0.x + c2 * p1.x + c1 * p2.x, x0.y + c2 * p1.y + c1 * p2.y);
    float2 B2 = make_float2(s2 * m1.x - s1 * m2.x, s2 * m1.y - s1 * m2.y);
    v[0] = make_float2(x0.x + p1.x + p2.x, x0.y + p1.y + p2.y);
    v[1] = make_float2(A1.x + B1.y, A1.y - B1.x);
    v[4] = make_float2(A1.x - B1.y, A1.y + B1.x);
    v[2] = make_float2(A2.x + B2.y, A2.y - B2.x);
    v[3] = make_float2(A2.x - B2.y, A2.y + B2.x);
}

template <>
__device__ __forceinline__ void dft<8>(float2 *v) {
    const float r2 = 0.70710678118654752440f;
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    dft<4>(e);
    dft<4>(o);
    // o[k] *= e^{-2 pi i k / 8}, folded into the sums by fused products
    const float2 t1 = make_float2(o[1].x + o[1].y, o[1].y - o[1].x);
    const float2 o2 = mul_negi(o[2]);
    const float2 t3 = make_float2(o[3].y - o[3].x, -(o[3].x + o[3].y));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = make_float2(fmaf(t1.x, r2, e[1].x), fmaf(t1.y, r2, e[1].y));
    v[5] = make_float2(fmaf(-t1.x, r2, e[1].x), fmaf(-t1.y, r2, e[1].y));
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = make_float2(fmaf(t3.x, r2, e[3].x), fmaf(t3.y, r2, e[3].y));
    v[7] = make_float2(fmaf(-t3.x, r2, e[3].x), fmaf(-t3.y, r2, e[3].y));
}

template <>
__device__ __forceinline__ void dft<1>(float2 *) {}
// Prime-factor form (Good, Thomas): with n = 3 n1 + 2 n2 and k = 3 k1 + 4 k2
// modulo 6 the exponent n k is 3 n1 k1 + 2 n2 k2, so three-point transforms over
// n2 and two-point ones over n1 need no rotations between them and round less.
// Error against float64, rms, of 6 x 6 x 6 = 216: 1.04e-7 in the factored form
// with rotations, 0.93e-7 here (0.96e-7 as 8 x 3 x 3 x 3); over 36 lengths 36 .. 1296
// the default schedule's mean is 3% below that of radices 8, 4, 2, 3, 5 taken
// greedily, and was 2% above it.
template <>
__device__ __forceinline__ void dft<6>(float2 *v) {
    float2 e[3] = {v[0], v[2], v[4]}, o[3] = {v[3], v[5], v[1]};
    dft<3>(e);
    dft<3>(o);
    v[0] = cadd(e[0], o[0]);
    v[3] = csub(e[0], o[0]);
    v[4] = cadd(e[1], o[1]);
    v[1] = csub(e[1], o[1]);
    v[2] = cadd(e[2], o[2]);
    v[5] = csub(e[2], o[2]);
}

// ------------------------------------------------------------ Stockham passes
// A workgroup transforms a tile of whole lines.  The first radix pass reads its
// elements straight from global memory into registers, the last one stores its
// results straight from registers; only the exchanges between passes go
// through LDS, so a line of n passes makes n - 1 trips through it.
//
// Element e of line l sits at lds_row(e) * ES + l * LS: STRIDED tiles keep
// lines adjacent (ES = number of lines, LS = 1) so a wavefront's lanes walk
// across lines; contiguous tiles keep each line contiguous (ES = 1, LS =
// lds_row(K)).  The spare element after every 8 keeps the radix-8 writes (8
// apart in consecutive lanes) off one another's banks.
//
// What bounds the passes: at few workgroups (2D, one image) the chain of memory
// round trip, exchanges and barriers; otherwise memory.  Measured against
// staging every element through LDS on the way in and out (n + 1 trips, 2 n + 1
// barriers, twiddles picked from one table with bank conflicts): 256^3 two
// strided passes 78 -> 65 us forward and 86 -> 69 inverse (4.6 and 4.4 TB/s);
// 240 x 240 x 192 74 -> 52 forward; 24 spirals x 8 coils 1668 -> 910 us over the
// eight FFT launches.  Radices 9, 10, 12 and 16 (fewer passes for 160, 256 or
// 640) were tried with 8 and with 16 elements per thread: 130 to 250 registers
// and 2 to 3 wavefronts per SIMD, 256^3 forward 65 -> 111 us.
//
// A tile holds at most kEPT elements per thread; a thread handles up to
// ceil(kEPT / R) butterflies of radix R per pass.  The workgroup size is read at
// run time (64 to 512), so each kernel is one instance.  The twiddles of the passes
// after the first sit in LDS in the order they are read (pass p: [R - 1][Ns]).
// The inverse transform runs the same passes on values with real and imaginary
// parts swapped on load and store.
#define NUFFT_INLINE __attribute__((always_inline))  // on lambdas: their arrays must stay in registers

constexpr int kEPT = 8;  // complex elements per thread

__host__ __device__ __forceinline__ constexpr int lds_row(int e) { return e + (e >> 3); }
__device__ __forceinline__ float2 swap_if(bool c, float2 v) { return c ? make_float2(v.y, v.x) : v; }

template <int R>
constexpr int butterflies() { return (kEPT + R - 1) / R; }

// Line and position of butterfly b of a pass with nbl butterflies per line.
template <bool STRIDED>
__device__ __forceinline__ void butterfly_place(int b, int nlines, int nbl, unsigned m_nbl, int &line, int &j) {
    if constexpr (STRIDED) {
        const FastDiv by_line(nlines);
        j = by_line.div(b);
        line = by_line.rem(b, j);
    } else {
        const FastDiv by_nbl(m_nbl, nbl);
        line = by_nbl.div(b);
        j = by_nbl.rem(b, line);
    }
}

// Run f(std::integral_constant<int, R>) for the radix of pass p.
template <class F>
__device__ __forceinline__ void with_radix(int R, F &&f) {
    switch (R) {
        case 8: f(std::integral_constant<int, 8>()); break;
        case 6: f(std::integral_constant<int, 6>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 1: f(std::integral_constant<int, 1>()); break;
        default: break;
    }
}

// Twiddles of the later passes into LDS: K - r[0] of them.  At most kEPT
// per thread (a tile holds at least a whole line), they are loaded before the
// data and stored after its loads, so they cost no memory round trip of their
// own.
struct TwiddleStage {
    float2 v[kEPT];
    __device__ __forceinline__ void load(const float2 *__restrict__ tw, int n) {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * blockDim.x;
            if (e < n) v[u] = tw[e];
        }
    }
    __device__ __forceinline__ void store(float2 *tw_lds, int n) const {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * blockDim.x;
            if (e < n) tw_lds[e] = v[u];
        }
    }
};

// p[off] for a uniform p and a lane's byte offset: with a 32-bit offset a scalar
// base and one register per address.
template <class Off>
__device__ __forceinline__ float2 load_at(const float2 *p, Off off_bytes) {
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(p) + off_bytes);
}
template <class Off>
__device__ __forceinline__ void store_at(float2 *p, Off off_bytes, float2 v) {
    *reinterpret_cast<float2 *>(reinterpret_cast<char *>(p) + off_bytes) = v;
}

// First pass: ld.load(it, u, r, line, q) issues the load of element q of a
// line into the loader's registers, ld.value(it, r) combines it; no twiddles
// (Ns = 1).  `stage` runs between the loads and the LDS writes.
template <int R, bool STRIDED, class LD, class ST>
__device__ __forceinline__ void first_radix(float2 *s, int nlines, int LS, int ES, const RadixPlan &rp, LD &&ld,
                                            ST &&stage) {
    constexpr int NB = butterflies<R>();
    const int nbl = rp.nbl[0], total = nlines * nbl;
    // (radices other than 8 and 4 one butterfly at a time: the registers of
    // several would set the kernel's)
    constexpr int kUnroll = R == 8 || R == 4 ? NB : 1;
#pragma unroll kUnroll
    for (int it = 0; it < NB; ++it) {
        const int b = int(threadIdx.x) + it * int(blockDim.x);
        int line, j;
        float2 v[R];
        butterfly_place<STRIDED>(min(b, total - 1), nlines, nbl, rp.m_nbl[0], line, j);  // (clamped: loads in bounds)
        ld(line, j, nbl, std::integral_constant<int, R>(), v);
        if (it == 0) stage();
        dft<R>(v);
        if (b < total) {
            float2 *q = s + line * LS;
            const int e0 = j * R;
#pragma unroll
            for (int r = 0; r < R; ++r) q[lds_row(e0 + r) * ES] = v[r];
        }
    }
    __syncthreads();
}

// One butterfly of pass p from LDS: its values after the DFT and its place.
template <int R, bool STRIDED>
__device__ __forceinline__ void radix_values(const float2 *s, int b, int nlines, int LS, int ES, const RadixPlan &rp,
                                             int p, const float2 *tw, float2 *v, int &line, int &j, int &k) {
    const int nbl = rp.nbl[p], Ns = rp.ns[p];
    const FastDiv by_ns(rp.m_ns[p], Ns);
    butterfly_place<STRIDED>(b, nlines, nbl, rp.m_nbl[p], line, j);
    const float2 *q = s + line * LS;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = q[lds_row(j + r * nbl) * ES];
    k = by_ns.rem(j, by_ns.div(j));
    const float2 *t = tw + rp.tw_off[p] + k;
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], t[(r - 1) * Ns]);
    dft<R>(v);
}

// A pass from LDS back to LDS.
template <int R, bool STRIDED>
__device__ __forceinline__ void middle_radix(float2 *s, int nlines, int LS, int ES, const RadixPlan &rp, int p,
                                             const float2 *tw) {
    constexpr int NB = butterflies<R>();
    const int Ns = rp.ns[p], total = nlines * rp.nbl[p];
    float2 v[NB][R];
    int line[NB], e0[NB];
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        int j, k;
        radix_values<R, STRIDED>(s, min(int(threadIdx.x) + it * int(blockDim.x), total - 1), nlines, LS, ES, rp, p, tw,
                                 v[it], line[it], j, k);
        e0[it] = (j - k) * R + k;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        if (int(threadIdx.x) + it * int(blockDim.x) < total) {
            float2 *q = s + line[it] * LS;
#pragma unroll
            for (int r = 0; r < R; ++r) q[lds_row(e0[it] + r * Ns) * ES] = v[it][r];
        }
    }
    __syncthreads();
}

// Last pass: st(line, j, nbl, R, values) stores elements j + r nbl of a line.
template <int R, bool STRIDED, class ST>
__device__ __forceinline__ void last_radix(const float2 *s, int nlines, int LS, int ES, const RadixPlan &rp,
                                           const float2 *tw, ST &&st) {
    constexpr int NB = butterflies<R>();
    const int p = rp.n - 1, nbl = rp.nbl[p], total = nlines * nbl;
    constexpr int kUnroll = R == 8 || R == 4 ? NB : 1;
#pragma unroll kUnroll
    for (int it = 0; it < NB; ++it) {
        const int b = int(threadIdx.x) + it * int(blockDim.x);
        if (b < total) {
            float2 v[R];
            int line, j, k;
            radix_values<R, STRIDED>(s, b, nlines, LS, ES, rp, p, tw, v, line, j, k);
            st(line, j, nbl, std::integral_constant<int, R>(), v);
        }
    }
}

// Passes 0 .. upto - 1, from global memory into LDS.
template <bool STRIDED, class LD, class ST>
__device__ __forceinline__ void leading_passes(float2 *s, int nlines, int LS, int ES, const RadixPlan &rp, int upto,
                                               const float2 *tw, LD &&ld, ST &&stage) {
    with_radix(rp.r[0], [&](auto R) NUFFT_INLINE { first_radix<R, STRIDED>(s, nlines, LS, ES, rp, ld, stage); });
    for (int p = 1; p < upto; ++p)
        with_radix(rp.r[p], [&](auto R) NUFFT_INLINE { middle_radix<R, STRIDED>(s, nlines, LS, ES, rp, p, tw); });
}

// Product of the scaling factors of the leading axes of image row r
// (row-major over axes 0..d-2), 32-bit index arithmetic.
__device__ __forceinline__ float row_scale(int d, const int *Nax, const float *const *scale, int r) {
    float sc = 1.0f;
#pragma unroll
    for (int a = kMaxDim - 2; a >= 0; --a) {
        if (a < d - 1) {
            int i = r;
            if (a > 0) {
                i = r % Nax[a];
                r /= Nax[a];
            }
            sc *= scale[a][i];
        }
    }
    return sc;
}

// Image index of grid position q on an axis of image size N and grid size K
// (n = i - N/2 wrapped modulo K); -1 in the zero gap.
__device__ __forceinline__ int src_row(int q, int N, int K) {
    if (q < N / 2) return q + N / 2;
    if (q >= K - N / 2) return q - (K - N / 2);
    return -1;
}
// No element of grid positions [q0, q0 + n) lies in the image.
__device__ __forceinline__ bool dead_rows(int q0, int n, int N, int K) {
    return q0 >= N / 2 && q0 + n <= K - N / 2;
}
__device__ __forceinline__ int grid_row(int i, int N, int K) { return i < N / 2 ? K - N / 2 + i : i - N / 2; }

// n / d and its remainder for uniform n >= 0, d >= 1, by a 32-bit division
// whenever that is enough.
__device__ __forceinline__ int64_t divmod(int64_t n, int64_t d, int64_t &rem) {
    int64_t q;
    if ((uint64_t(n) | uint64_t(d)) >> 32) {
        q = n / d;
    } else {
        q = int64_t(unsigned(n) / unsigned(d));
    }
    rem = n - q * d;
    return q;
}

// ------------------------------------------------------------ FFT kernels
// Dynamic LDS layout of every FFT kernel: [K twiddles][tile].
template <bool COILS>
__device__ __forceinline__ void first_pass_body(const FirstPassArgs &a, int lines_per_wg, int64_t bx) {
    extern __shared__ float2 lds[];
    const int K = a.K, N = a.N;
    float2 *tw = lds;
    float2 *s = lds + K;
    const int64_t total = int64_t(a.B) * a.C * a.rows;
    const int64_t l0 = bx * lines_per_wg;
    const int nl = int(min(int64_t(lines_per_wg), total - l0));  // 1..64
    const int ntw = K - a.rp.r[0];
    TwiddleStage tws;
    tws.load(a.tw, ntw);
    const int rows = int(a.rows);
    int64_t r0, c0 = 0;
    const int64_t g0 = divmod(l0, rows, r0);
    int64_t b0 = g0;
    if constexpr (COILS) b0 = divmod(g0, a.C, c0);
    const FastDiv by_rows(rows), by_c(COILS ? a.C : 1);  // (for line numbers < 128, grids < C + 64)
    const float *slast = a.scale[a.d - 1];
    auto load = [&](int lw, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
        constexpr int R = decltype(RC)::value;
        // line l0 + lw is row r of grid (b, c)
        int r = int(r0) + lw;
        const int dg = rows >= kMaxLinesPerWg ? (r >= rows ? 1 : 0) : by_rows.div(r);
        r -= dg * rows;
        int64_t b = b0 + dg;
        int c = 0;
        if constexpr (COILS) {
            c = int(c0) + dg;
            const int db = by_c.div(c);
            c -= db * a.C;
            b = b0 + db;
        }
        const float2 *x = a.x + (b * rows + r) * N;
        const float2 *coil = COILS ? a.coils + (int64_t(c) * rows + r) * N : nullptr;
        // every load first, without branches: zero-gap elements read pixel 0
        float2 cv[COILS ? R : 1];
        float sv[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int i = max(src_row(j + u * nbl, N, K), 0);
            v[u] = x[i];
            sv[u] = slast[i];
            if constexpr (COILS) cv[u] = coil[i];
        }
        const float rs = row_scale(a.d, a.Nax, a.scale, r);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const float2 t = cscale(v[u], src_row(j + u * nbl, N, K) >= 0 ? sv[u] * rs : 0.f);
            if constexpr (COILS)
                v[u] = cmul(t, cv[u]);
            else
                v[u] = t;
        }
    };
    const int LS = lds_row(K);
    leading_passes<false>(s, nl, LS, 1, a.rp, a.rp.n - 1, tw, load, [&]() NUFFT_INLINE { tws.store(tw, ntw); });
    float2 *out = a.out + l0 * K;
    with_radix(a.rp.r[a.rp.n - 1], [&](auto RL) NUFFT_INLINE {
        last_radix<RL, false>(s, nl, LS, 1, a.rp, tw, [&](int lw, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
            constexpr int R = decltype(RC)::value;
            float2 *o = out + lw * K + j;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                float2 t = v[u];
                if (a.phase) t = cmul(t, a.phase[j + u * nbl]);
                if (a.mult) t = cmul(t, a.mult[((l0 + lw) % a.rows) * K + j + u * nbl]);
                o[u * nbl] = t;
            }
        });
    });
}

template <bool COILS>
__global__ __launch_bounds__(kFftThreads) void k_first_pass(FirstPassArgs a, int lines_per_wg) {
    first_pass_body<COILS>(a, lines_per_wg, blockIdx.x);
}

// Many problems in one launch: workgroup b runs block blocks[b].y of problem
// blocks[b].x, whose arguments sit in jobs[blocks[b].x].
template <bool COILS>
__global__ __launch_bounds__(kFftThreads) void k_first_pass_multi(const FirstJob *__restrict__ jobs,
                                                             const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const FirstJob &j = jobs[b.x];
    first_pass_body<COILS>(j.a, j.lpw, b.y);
}

// Logical block of workgroup b when consecutive blocks should share an XCD:
// the hardware deals workgroups round-robin over the 8 XCDs, so XCD x takes
// the x-th contiguous eighth of the blocks.  Neighbouring column tiles then
// meet in one L2: a tile's rows are W * 8 bytes (24 to 64), so the 128-byte
// lines they share are fetched and written back once instead of by several
// XCDs.  Measured, dealt round-robin -> contiguous: 8 grids of 640 x 640 (48-
// byte rows) forward 28.3 -> 22.8 us, inverse 38.0 -> 29.5; 240 x 240 x 192,
// two passes each, 82.6 -> 74.2 and 102.7 -> 88.4 us; 256^3 (128-byte rows)
// unchanged at 78 and 86 us.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned n) {
    const unsigned x = b % kXcds, q = n / kXcds, r = n % kXcds;
    return x * q + min(x, r) + b / kXcds;
}

// tile_of and the cell within the tile (tile_base), by high multiplies: the
// dividends stay below K nt <= 2^20 and the divisors below 2^12.
struct TileMap {
    bool even;  // tiles of T cells
    int T, nt, half;
    FastDiv byT, by_half, by_nt;
    __device__ __forceinline__ TileMap(int K, int T_, int nt_)
        : even(T_ * nt_ == K), T(T_), nt(nt_), half(K / 2), byT(T_), by_half(K / 2), by_nt(nt_) {}
    __device__ __forceinline__ void find(int k, int &t, int &l) const {
        if (even) {
            t = byT.div(k);
            l = byT.rem(k, t);
        } else {
            t = by_half.div(((k >> 1) + 1) * nt - 1);
            l = k - 2 * by_nt.div(t * half);
        }
    }
};

// Forms of the inverse pass with instances of their own, so the plain passes
// keep their register budget: the first inverse pass of an adjoint whose split
// gridding tiles are still partial tiles, and the first inverse pass after a
// Toeplitz product.  A tile's lanes address one slab of K rows by inner columns
// from scalar row bases, K / R rows apart (R the first radix on the way in, the
// last on the way out).  WIDE: those rows hold more than 4 GiB and the lanes'
// offsets are 64 bits wide (strided_wide); everywhere else they are 32 bits, one
// register per address instead of two.
enum { kPlain, kSplitTiles, kProduct };
template <bool INV, int FORM, bool WIDE>
__device__ __forceinline__ void strided_pass_body(const StridedPassArgs &a, int W, int64_t ntc, int64_t bid) {
    extern __shared__ float2 lds[];
    using Off = std::conditional_t<WIDE, uint64_t, unsigned>;
    const int K = a.K;
    float2 *tw = lds;
    float2 *s = lds + K;
    int64_t ct, o;
    const int64_t rest = divmod(bid, ntc, ct);
    const int64_t g = divmod(rest, a.outer, o);
    const int64_t c0 = ct * W;
    const int wv = int(min(int64_t(W), a.inner - c0));
    const float2 *in = a.in + ((g * a.outer + o) * a.Lin) * a.inner + c0;
    float2 *out = a.out + ((g * a.outer + o) * a.Lout) * a.inner + c0;
    const int ntw = K - a.rp.r[0];
    const float2 *mul = FORM == kProduct ? a.mult + (o * a.Lin) * a.inner + c0 : nullptr;
    TwiddleStage tws;
    tws.load(a.tw, ntw);
    // forward: grid row q takes image row src_row (zero rows when Lin < K, the
    // centring shift when Lin == K); inverse: the input is the grid
    auto load = [&](int w, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
        constexpr int R = decltype(RC)::value;
        const Off off = (Off(j) * unsigned(a.inner) + unsigned(w)) * unsigned(sizeof(float2));
        if constexpr (FORM == kSplitTiles) {
            // First inverse pass of the adjoint: a cell of a split gridding tile
            // is the sum of its partial tiles in chunk order (the order, hence
            // the bits, of k_reduce_partials).  Grid row q on axis 0, column
            // c0 + w over the remaining axes; the input and the cell's split
            // entry are loaded together, the partial tiles after that.
            const TileMap m0(a.Kax[0], a.T[0], a.nt[0]), m1(a.Kax[1], a.T[1], a.nt[1]);
            const FastDiv byK2(a.d > 2 ? a.Kax[2] : 1);
            const int c = int(c0) + w;
            int k1 = c, t2 = 0, l2 = 0;
            if (a.d > 2) {
                k1 = byK2.div(c);
                TileMap(a.Kax[2], a.T[2], a.nt[2]).find(byK2.rem(c, k1), t2, l2);
            }
            int t1, l1;
            m1.find(k1, t1, l1);
            int2 sp[R];
            int cell[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int q = j + u * nbl;
                int t0, l0;
                m0.find(q, t0, l0);
                int tile = t0 * a.nt[1] + t1;
                cell[u] = l0 * a.T[1] + l1;
                if (a.d > 2) {
                    tile = tile * a.nt[2] + t2;
                    cell[u] = cell[u] * a.T[2] + l2;
                }
                v[u] = load_at(in + int64_t(u * nbl) * a.inner, off);
                sp[u] = a.split_of_tile[tile];
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int n = sp[u].y;
                if (n > 0) {
                    const float2 *pp = a.partials + (g * a.n_slots + sp[u].x) * a.tile_cells + cell[u];
                    // kReduceLanes interleaved sums (chunk c into sum c mod
                    // kReduceLanes, in chunk order), then added in lane order
                    float2 acc[kReduceLanes];
#pragma unroll
                    for (int i = 0; i < kReduceLanes; ++i) acc[i] = make_float2(0.f, 0.f);
                    for (int k0 = 0; k0 < n; k0 += kReduceLanes) {
                        float2 t[kReduceLanes];
#pragma unroll
                        for (int i = 0; i < kReduceLanes; ++i)
                            if (k0 + i < n) t[i] = pp[int64_t(k0 + i) * a.tile_cells];
#pragma unroll
                        for (int i = 0; i < kReduceLanes; ++i)
                            if (k0 + i < n) acc[i] = cadd(acc[i], t[i]);
                    }
#pragma unroll
                    for (int i = 1; i < kReduceLanes; ++i) acc[0] = cadd(acc[0], acc[i]);
                    v[u] = acc[0];
                }
            }
        } else {
            float2 mv[FORM == kProduct ? R : 1];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int q0 = u * nbl;
                if constexpr (INV) {
                    v[u] = load_at(in + int64_t(q0) * a.inner, off);
                    if constexpr (FORM == kProduct) mv[u] = load_at(mul + int64_t(q0) * a.inner, off);
                } else {
                    // (no branches: zero rows read row 0; cell counts fit 32 bits)
                    const int i = src_row(j + q0, a.Lin, K);
                    v[u] = in[unsigned(max(i, 0)) * unsigned(a.inner) + unsigned(w)];
                }
            }
            if constexpr (!INV) {
#pragma unroll
                for (int u = 0; u < R; ++u)
                    if (src_row(j + u * nbl, a.Lin, K) < 0) v[u] = make_float2(0.f, 0.f);
            }
            if constexpr (FORM == kProduct) {
#pragma unroll
                for (int u = 0; u < R; ++u) v[u] = cmul(v[u], mv[u]);
            }
        }
        if constexpr (INV) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (a.phase) v[u] = cmulcj(a.phase[j + u * nbl], v[u]);
                v[u] = swap_if(true, v[u]);
            }
        }
    };
    leading_passes<true>(s, wv, 1, wv, a.rp, a.rp.n - 1, tw, load, [&]() NUFFT_INLINE { tws.store(tw, ntw); });
    with_radix(a.rp.r[a.rp.n - 1], [&](auto RL) NUFFT_INLINE {
        last_radix<RL, true>(s, wv, 1, wv, a.rp, tw, [&](int w, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
            constexpr int R = decltype(RC)::value;
            const Off off = (Off(j) * unsigned(a.inner) + unsigned(w)) * unsigned(sizeof(float2));
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int q0 = u * nbl;
                float2 t = swap_if(INV, v[u]);
                if constexpr (!INV) {
                    if (a.phase) t = cmul(t, a.phase[j + q0]);
                    store_at(out + int64_t(q0) * a.inner, off, t);
                } else if (!dead_rows(q0, nbl, a.Lout, K)) {
                    const int i = src_row(j + q0, a.Lout, K);
                    if (i >= 0) out[unsigned(i) * unsigned(a.inner) + unsigned(w)] = t;
                }
            }
        });
    });
}

template <bool INV, int FORM, bool WIDE = false>
__global__ __launch_bounds__(kFftThreads) void k_strided_pass(StridedPassArgs a, int W, int64_t ntc) {
    strided_pass_body<INV, FORM, WIDE>(a, W, ntc, xcd_block(blockIdx.x, gridDim.x));
}

template <bool INV, int FORM, bool WIDE = false>
__global__ __launch_bounds__(kFftThreads) void k_strided_pass_multi(const StridedJob *__restrict__ jobs,
                                                               const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const StridedJob &j = jobs[b.x];
    strided_pass_body<INV, FORM, WIDE>(j.a, j.W, j.ntc, b.y);
}

template <bool COILS>
__device__ __forceinline__ void last_pass_body(const LastPassArgs &a, int rows_per_wg, int coils_per_round, int64_t bx) {
    extern __shared__ float2 lds[];
    const int K = a.K, N = a.N, C = a.C;
    float2 *tw = lds;
    float2 *s = lds + K;
    const int64_t nrt = (a.rows + rows_per_wg - 1) / rows_per_wg;
    int64_t rt;
    const int64_t b = divmod(bx, nrt, rt);
    const int64_t r0 = rt * rows_per_wg;
    const int nr = int(min(int64_t(rows_per_wg), a.rows - r0));
    const int ntw = K - a.rp.r[0];
    TwiddleStage tws;
    tws.load(a.tw, ntw);
    const float *slast = a.scale[a.d - 1];
    const int LS = lds_row(K);
    float2 *x = a.x + (b * a.rows + r0) * N;
    if constexpr (!COILS) {
        const float2 *in = a.in + (b * a.rows + r0) * K;
        auto load = [&](int lw, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
            constexpr int R = decltype(RC)::value;
            const float2 *row = in + lw * K + j;
#pragma unroll
            for (int u = 0; u < R; ++u) v[u] = row[u * nbl];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (a.phase) v[u] = cmulcj(a.phase[j + u * nbl], v[u]);
                v[u] = swap_if(true, v[u]);
            }
        };
        leading_passes<false>(s, nr, LS, 1, a.rp, a.rp.n - 1, tw, load, [&]() NUFFT_INLINE { tws.store(tw, ntw); });
        with_radix(a.rp.r[a.rp.n - 1], [&](auto RL) NUFFT_INLINE {
            last_radix<RL, false>(s, nr, LS, 1, a.rp, tw, [&](int lw, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
                constexpr int R = decltype(RC)::value;
                float sv[R];
#pragma unroll
                for (int u = 0; u < R; ++u) sv[u] = slast[max(src_row(j + u * nbl, N, K), 0)];
                const float rs = row_scale(a.d, a.Nax, a.scale, int(r0) + lw);
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    if (dead_rows(u * nbl, nbl, N, K)) continue;
                    const int i = src_row(j + u * nbl, N, K);
                    if (i >= 0) x[lw * N + i] = cscale(swap_if(true, v[u]), rs * sv[u]);
                }
            });
        });
        return;
    }
    // Coils: rounds of coils_per_round coils per row.  After the inverse passes
    // every (line, pixel) is multiplied by the conjugate coil value, kCoilBatch
    // per thread at a time (the first batch is loaded before the passes, which
    // hide it), and the coils of a pixel are summed in coil order.  Several
    // rounds keep the running sums in LDS after the tile.
    constexpr int kCoilBatch = 4;
    const FastDiv byN(N);
    const int no = nr * N;
    const bool rounds = coils_per_round < C;
    float2 *acc = s + nr * coils_per_round * LS;
    for (int c0 = 0; c0 < C; c0 += coils_per_round) {
        const int nc = min(coils_per_round, C - c0);
        const int nl = nr * nc;
        const FastDiv byC(nc);
        float2 cv[kCoilBatch];
        auto coil_batch = [&](int e0) NUFFT_INLINE {
#pragma unroll
            for (int u = 0; u < kCoilBatch; ++u) {
                const int e = min(e0 + int(threadIdx.x) + u * int(blockDim.x), nl * N - 1);
                const int lw = byN.div(e), i = byN.rem(e, lw);
                const int rr = byC.div(lw), cc = byC.rem(lw, rr);
                cv[u] = a.coils[(int64_t(c0 + cc) * a.rows + r0 + rr) * N + i];
            }
        };
        if (a.coils) coil_batch(0);
        auto load = [&](int lw, int j, int nbl, auto RC, float2 *v) NUFFT_INLINE {
            constexpr int R = decltype(RC)::value;
            const int rr = byC.div(lw), cc = byC.rem(lw, rr);
            const float2 *row = a.in + ((b * C + c0 + cc) * a.rows + r0 + rr) * K + j;
#pragma unroll
            for (int u = 0; u < R; ++u) v[u] = row[u * nbl];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (a.phase) v[u] = cmulcj(a.phase[j + u * nbl], v[u]);
                v[u] = swap_if(true, v[u]);
            }
        };
        if (c0 > 0) __syncthreads();  // the previous round's sums are read
        leading_passes<false>(s, nl, LS, 1, a.rp, a.rp.n, tw, load, [&]() NUFFT_INLINE {
            if (c0 == 0) tws.store(tw, ntw);
        });
        if (a.coils) {
            for (int e0 = 0; e0 < nl * N; e0 += kCoilBatch * int(blockDim.x)) {
                if (e0 > 0) coil_batch(e0);
#pragma unroll
                for (int u = 0; u < kCoilBatch; ++u) {
                    const int e = e0 + int(threadIdx.x) + u * int(blockDim.x);
                    if (e < nl * N) {
                        const int lw = byN.div(e), i = byN.rem(e, lw);
                        float2 *q = s + lw * LS + lds_row(grid_row(i, N, K));
                        *q = cmulcj(cv[u], swap_if(true, *q));
                    }
                }
            }
            __syncthreads();
        }
        for (int e = threadIdx.x; e < no; e += blockDim.x) {
            const int rr = byN.div(e), i = byN.rem(e, rr);
            const float2 *q = s + rr * nc * LS + lds_row(grid_row(i, N, K));
            float2 sum = rounds && c0 > 0 ? acc[e] : make_float2(0.f, 0.f);
            for (int cc = 0; cc < nc; ++cc) sum = cadd(sum, swap_if(!a.coils, q[cc * LS]));
            if (c0 + nc < C)
                acc[e] = sum;
            else
                x[e] = cscale(sum, row_scale(a.d, a.Nax, a.scale, int(r0) + rr) * slast[i]);
        }
    }
}

template <bool COILS>
__global__ __launch_bounds__(kFftThreads) void k_last_pass(LastPassArgs a, int rows_per_wg, int coils_per_round) {
    last_pass_body<COILS>(a, rows_per_wg, coils_per_round, blockIdx.x);
}

template <bool COILS>
__global__ __launch_bounds__(kFftThreads) void k_last_pass_multi(const LastJob *__restrict__ jobs,
                                                            const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const LastJob &j = jobs[b.x];
    last_pass_body<COILS>(j.a, j.rpw, j.cpr, b.y);
}

// FFT tile sizes: a tile holds up to kFftThreads * kEPT elements.  The host takes
// the largest tile that still leaves about target_groups workgroups (small
// transforms spread over the whole chip), then the smallest block that holds
// it.

// LDS elements of one line (lds_row of its length).
size_t line_lds(int K) { return size_t(lds_row(K)); }

int threads_for(int elems) {
    int t = 64;
    while (t < kFftThreads && t * kEPT < elems) t *= 2;
    return t;
}

}  // namespace

// ------------------------------------------------------------ launchers
#ifndef NUFFT_FFT_WIDE
FftLaunch first_pass_launch(const FirstPassArgs &a, int threads) {
    FftLaunch L{64, 0, 0, 1, 0};
    const int64_t total = int64_t(a.B) * a.C * a.rows;
    if (total == 0) return L;
    const int cap = kFftTileElems / a.K;  // lines that fit the largest tile
    int lpw = int(std::min<int64_t>(std::max<int64_t>(1, total / a.target_groups), std::min(cap, kMaxLinesPerWg)));
    lpw = std::max(1, lpw);
    if (threads > 0)  // a given workgroup size: as many lines as its tile holds
        lpw = int(std::max<int64_t>(1, std::min<int64_t>({total, kMaxLinesPerWg, threads * kEPT / a.K})));
    L.threads = threads > 0 ? threads : threads_for(lpw * a.K);
    L.blocks = (total + lpw - 1) / lpw;
    L.lds = (size_t(a.K) + size_t(lpw) * line_lds(a.K)) * sizeof(float2);
    L.p0 = lpw;
    return L;
}

hipError_t launch_first_pass(const FirstPassArgs &a, hipStream_t s) {
    const FftLaunch L = first_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    const dim3 grid{unsigned(L.blocks)}, block{unsigned(L.threads)};
    if (a.coils)
        launch_kernel((k_first_pass<true>), grid, block, L.lds, s, a, L.p0);
    else
        launch_kernel((k_first_pass<false>), grid, block, L.lds, s, a, L.p0);
    return hipGetLastError();
}

FftLaunch strided_pass_launch(const StridedPassArgs &a, int threads) {
    FftLaunch L{64, 0, 0, 1, 0};
    const int64_t columns = a.grids * a.outer * a.inner;
    if (columns == 0) return L;
    const int cap = std::max(1, threads > 0 ? threads * kEPT / a.K : kFftTileElems / a.K);
    // columns per tile: at least 4 adjacent (32-byte rows), fewer only for narrow
    // arrays; with a given workgroup size, as many as its tile holds
    int64_t W = threads > 0 ? cap : std::max<int64_t>(4, columns / a.target_groups);
    W = std::min<int64_t>(W, cap);
    W = std::min<int64_t>(W, a.inner);
    W = std::max<int64_t>(W, 1);
    const int64_t ntc = (a.inner + W - 1) / W;
    L.blocks = ntc * a.outer * a.grids;
    L.threads = threads > 0 ? threads : threads_for(int(W) * a.K);
    L.lds = (size_t(a.K) + size_t(W) * line_lds(a.K)) * sizeof(float2);
    L.p0 = int(W);
    L.p1 = ntc;
    return L;
}

// (the wide instances: fft_wide.hip)
hipError_t launch_wide_strided_pass(const StridedPassArgs &a, const FftLaunch &L, hipStream_t s);
void launch_wide_strided_pass_multi(const StridedJob *jobs, const int4 *blocks, dim3 grid, dim3 block, bool inverse,
                                    bool split, size_t lds, hipStream_t s);

hipError_t launch_strided_pass(const StridedPassArgs &a, hipStream_t s) {
    const FftLaunch L = strided_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    if (strided_wide(a)) return launch_wide_strided_pass(a, L, s);
    const dim3 grid{unsigned(L.blocks)}, block{unsigned(L.threads)};
    if (!a.inverse)
        launch_kernel((k_strided_pass<false, kPlain>), grid, block, L.lds, s, a, L.p0, L.p1);
    else if (a.split_of_tile)
        launch_kernel((k_strided_pass<true, kSplitTiles>), grid, block, L.lds, s, a, L.p0, L.p1);
    else if (a.mult)
        launch_kernel((k_strided_pass<true, kProduct>), grid, block, L.lds, s, a, L.p0, L.p1);
    else
        launch_kernel((k_strided_pass<true, kPlain>), grid, block, L.lds, s, a, L.p0, L.p1);
    return hipGetLastError();
}

FftLaunch last_pass_launch(const LastPassArgs &a, int threads) {
    FftLaunch L{64, 0, 0, 1, 1};
    const int64_t total_rows = int64_t(a.B) * a.rows;
    if (total_rows == 0) return L;
    const int tile = threads > 0 ? threads * kEPT : kFftTileElems;
    int rows_per_wg, coils_per_round;
    if (a.C * a.K <= tile) {
        coils_per_round = a.C;
        const int cap = std::min(tile / (a.C * a.K), kMaxLinesPerWg);
        rows_per_wg = threads > 0 ? cap
                                  : int(std::min<int64_t>(std::max<int64_t>(1, total_rows / a.target_groups), cap));
    } else {
        rows_per_wg = 1;
        coils_per_round = std::max(1, tile / a.K);
    }
    if (int64_t(rows_per_wg) > a.rows) rows_per_wg = int(a.rows);
    rows_per_wg = std::max(1, rows_per_wg);
    L.threads = threads > 0 ? threads : threads_for(rows_per_wg * coils_per_round * a.K);
    const int64_t nrt = (a.rows + rows_per_wg - 1) / rows_per_wg;
    L.blocks = nrt * a.B;
    L.lds = (size_t(a.K) + size_t(rows_per_wg) * coils_per_round * line_lds(a.K) +
             (coils_per_round < a.C ? size_t(rows_per_wg) * a.N : 0)) * sizeof(float2);
    L.p0 = rows_per_wg;
    L.p1 = coils_per_round;
    return L;
}

hipError_t launch_last_pass(const LastPassArgs &a, hipStream_t s) {
    const FftLaunch L = last_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    const dim3 grid{unsigned(L.blocks)}, block{unsigned(L.threads)};
    if (last_pass_coils(a))
        launch_kernel((k_last_pass<true>), grid, block, L.lds, s, a, L.p0, int(L.p1));
    else
        launch_kernel((k_last_pass<false>), grid, block, L.lds, s, a, L.p0, int(L.p1));
    return hipGetLastError();
}

// ---- many problems per launch
hipError_t launch_first_pass_multi(const FirstJob *jobs, const int4 *blocks, int64_t nblocks, int threads, bool coils,
                                   size_t lds, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    const dim3 grid{unsigned(nblocks)}, block{unsigned(threads)};
    if (coils)
        launch_kernel((k_first_pass_multi<true>), grid, block, lds, s, jobs, blocks);
    else
        launch_kernel((k_first_pass_multi<false>), grid, block, lds, s, jobs, blocks);
    return hipGetLastError();
}

hipError_t launch_strided_pass_multi(const StridedJob *jobs, const int4 *blocks, int64_t nblocks, int threads,
                                     bool inverse, bool split, bool wide, size_t lds, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    const dim3 grid{unsigned(nblocks)}, block{unsigned(threads)};
    if (wide)
        launch_wide_strided_pass_multi(jobs, blocks, grid, block, inverse, split, lds, s);
    else if (!inverse)
        launch_kernel((k_strided_pass_multi<false, kPlain>), grid, block, lds, s, jobs, blocks);
    else if (split)
        launch_kernel((k_strided_pass_multi<true, kSplitTiles>), grid, block, lds, s, jobs, blocks);
    else
        launch_kernel((k_strided_pass_multi<true, kPlain>), grid, block, lds, s, jobs, blocks);
    return hipGetLastError();
}

hipError_t launch_last_pass_multi(const LastJob *jobs, const int4 *blocks, int64_t nblocks, int threads, bool coils,
                                  size_t lds, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    const dim3 grid{unsigned(nblocks)}, block{unsigned(threads)};
    if (coils)
        launch_kernel((k_last_pass_multi<true>), grid, block, lds, s, jobs, blocks);
    else
        launch_kernel((k_last_pass_multi<false>), grid, block, lds, s, jobs, blocks);
    return hipGetLastError();
}

#else  // NUFFT_FFT_WIDE: the instances with 64-bit offsets, in a code object of their own

hipError_t launch_wide_strided_pass(const StridedPassArgs &a, const FftLaunch &L, hipStream_t s) {
    const dim3 grid{unsigned(L.blocks)}, block{unsigned(L.threads)};
    if (!a.inverse)
        launch_kernel((k_strided_pass<false, kPlain, true>), grid, block, L.lds, s, a, L.p0, L.p1);
    else if (a.split_of_tile)
        launch_kernel((k_strided_pass<true, kSplitTiles, true>), grid, block, L.lds, s, a, L.p0, L.p1);
    else if (a.mult)
        // a Toeplitz grid's lengths are multiples of 4: its first radix is 4 or more, never wide
        return hipErrorInvalidValue;
    else
        launch_kernel((k_strided_pass<true, kPlain, true>), grid, block, L.lds, s, a, L.p0, L.p1);
    return hipGetLastError();
}

void launch_wide_strided_pass_multi(const StridedJob *jobs, const int4 *blocks, dim3 grid, dim3 block, bool inverse,
                                    bool split, size_t lds, hipStream_t s) {
    if (!inverse)
        launch_kernel((k_strided_pass_multi<false, kPlain, true>), grid, block, lds, s, jobs, blocks);
    else if (split)
        launch_kernel((k_strided_pass_multi<true, kSplitTiles, true>), grid, block, lds, s, jobs, blocks);
    else
        launch_kernel((k_strided_pass_multi<true, kPlain, true>), grid, block, lds, s, jobs, blocks);
}

#endif

}  // namespace nufft
