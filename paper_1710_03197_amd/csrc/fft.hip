// FFT kernels of the pair (paper Section 2.1 "Oversampled FFT"):
//   k_first_pass   S + zero padding + FFT along the contiguous last axis
//                  (Section 2.1 "Scaling", "Oversampled FFT"); the pad is index
//                  arithmetic on the load, never a materialised array.
//   k_strided_pass FFT along a strided axis, zero-padded input rows (forward) or
//                  cropped output rows (adjoint, the copy after the IFFT).
//   k_last_pass    inverse FFT along the last axis + crop + S^H + coil combine
//                  (Section 2.2, multi-coil: sum_i conj(c_i) A^H y_i).
// All arithmetic is float32.
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
    // o[k] *= e^{-2 pi i k / 8}
    float2 o1 = make_float2((o[1].x + o[1].y) * r2, (o[1].y - o[1].x) * r2);
    float2 o2 = mul_negi(o[2]);
    float2 o3 = make_float2((o[3].y - o[3].x) * r2, -(o[3].x + o[3].y) * r2);
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
}

// ------------------------------------------------------------ Stockham passes in LDS
// Element (line, q) of a tile lives at s[line * LS + q * ES].  STRIDED tiles
// keep lines adjacent (ES = number of lines) so a wavefront's lanes walk
// across lines; contiguous tiles keep each line contiguous (ES = 1).  A tile
// holds at most THREADS * kEPT complex elements; a thread handles up to
// ceil(kEPT / R) butterflies of radix R per pass.  Twiddles e^{-2 pi i e / K}
// are staged in LDS (tw) once per workgroup.
constexpr int kEPT = 8;  // complex elements per thread

// KC > 0: the line length KC and sub-transform length NSC of this pass are
// compile-time constants (the common grid sizes), so its index arithmetic
// folds; the same operations in the same order as the run-time form.
template <int THREADS, int R, bool INV, bool STRIDED, int KC = 0, int NSC = 0>
__device__ __forceinline__ void radix_pass(float2 *s, int nlines, int K_, int LS, int ES, int Ns_, int span_,
                                           unsigned m_ns, unsigned m_nbl, const float2 *tw) {
    constexpr int NB = (kEPT + R - 1) / R;
    const int K = KC > 0 ? KC : K_;
    const int Ns = KC > 0 ? NSC : Ns_;
    const int span = KC > 0 ? KC / ((NSC > 0 ? NSC : 1) * R) : span_;
    const int nbl = K / R;
    const int total = nlines * nbl;
    // (the line count's magic is made per pass: kept across passes it costs
    // the strided passes about 20 registers)
    const FastDiv by_line = STRIDED ? FastDiv(nlines) : FastDiv(m_nbl, nbl), by_ns(m_ns, Ns);
    float2 v[NB][R];
    int lidx[NB], jidx[NB];
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        const int b = threadIdx.x + it * THREADS;
        lidx[it] = 0;
        jidx[it] = 0;
        if (b < total) {
            int line, j;
            if (STRIDED) {
                j = by_line.div(b);
                line = by_line.rem(b, j);
            } else if constexpr (KC > 0) {
                line = b / (KC / R);
                j = b - line * (KC / R);
            } else {
                line = by_line.div(b);
                j = by_line.rem(b, line);
            }
            lidx[it] = line;
            jidx[it] = j;
            const float2 *p = s + line * LS + j * ES;
#pragma unroll
            for (int r = 0; r < R; ++r) v[it][r] = p[r * nbl * ES];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        const int b = threadIdx.x + it * THREADS;
        if (b < total) {
            const int j = jidx[it];
            int jq, k;
            if constexpr (KC > 0) {
                jq = j / NSC;
                k = j - jq * NSC;
            } else {
                jq = by_ns.div(j);
                k = by_ns.rem(j, jq);
            }
            const int step = __umul24(k, span);
#pragma unroll
            for (int r = 1; r < R; ++r) {
                float2 w = tw[r * step];
                if (INV) w.y = -w.y;
                v[it][r] = cmul(v[it][r], w);
            }
            if (INV) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[it][r].y = -v[it][r].y;
            }
            dft<R>(v[it]);
            if (INV) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[it][r].y = -v[it][r].y;
            }
            const int idxD = __umul24(jq, Ns * R) + k;
            float2 *q = s + lidx[it] * LS + idxD * ES;
#pragma unroll
            for (int r = 0; r < R; ++r) q[r * Ns * ES] = v[it][r];
        }
    }
    __syncthreads();
}

template <int THREADS, bool INV, bool STRIDED>
__device__ void lds_fft(float2 *s, int nlines, int K, int LS, int ES, const RadixPlan &rp, const float2 *tw) {
    // the grid sizes of the common workloads (and their Toeplitz 2N grids)
    // with their radix plans spelled out at compile time
    if (K == 512 && rp.n == 3 && rp.r[0] == 8 && rp.r[1] == 8 && rp.r[2] == 8) {
        radix_pass<THREADS, 8, INV, STRIDED, 512, 1>(s, nlines, K, LS, ES, 1, 0, 0u, 0u, tw);
        radix_pass<THREADS, 8, INV, STRIDED, 512, 8>(s, nlines, K, LS, ES, 8, 0, 0u, 0u, tw);
        radix_pass<THREADS, 8, INV, STRIDED, 512, 64>(s, nlines, K, LS, ES, 64, 0, 0u, 0u, tw);
        return;
    }
    if (K == 256 && rp.n == 3 && rp.r[0] == 8 && rp.r[1] == 8 && rp.r[2] == 4) {
        radix_pass<THREADS, 8, INV, STRIDED, 256, 1>(s, nlines, K, LS, ES, 1, 0, 0u, 0u, tw);
        radix_pass<THREADS, 8, INV, STRIDED, 256, 8>(s, nlines, K, LS, ES, 8, 0, 0u, 0u, tw);
        radix_pass<THREADS, 4, INV, STRIDED, 256, 64>(s, nlines, K, LS, ES, 64, 0, 0u, 0u, tw);
        return;
    }
    int Ns = 1;
    for (int p = 0; p < rp.n; ++p) {
        const int R = rp.r[p];
        const int sp = rp.span[p];
        const unsigned mn = rp.m_ns[p], mb = rp.m_nbl[p];
        switch (R) {
            case 8: radix_pass<THREADS, 8, INV, STRIDED>(s, nlines, K, LS, ES, Ns, sp, mn, mb, tw); break;
            case 4: radix_pass<THREADS, 4, INV, STRIDED>(s, nlines, K, LS, ES, Ns, sp, mn, mb, tw); break;
            case 2: radix_pass<THREADS, 2, INV, STRIDED>(s, nlines, K, LS, ES, Ns, sp, mn, mb, tw); break;
            case 3: radix_pass<THREADS, 3, INV, STRIDED>(s, nlines, K, LS, ES, Ns, sp, mn, mb, tw); break;
            case 5: radix_pass<THREADS, 5, INV, STRIDED>(s, nlines, K, LS, ES, Ns, sp, mn, mb, tw); break;
            default: break;
        }
        Ns *= R;
    }
}

// Twiddles into LDS.  A workgroup's tile holds at least one whole line, so a
// thread stages at most kEPT of the K twiddles; every load is issued before
// the first LDS write, so the staging costs one memory round trip.
template <int THREADS>
struct TwiddleStage {
    float2 v[kEPT];
    __device__ __forceinline__ void load(const float2 *__restrict__ tw, int K) {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * THREADS;
            if (e < K) v[u] = tw[e];
        }
    }
    __device__ __forceinline__ void store(float2 *tw_lds, int K) const {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * THREADS;
            if (e < K) tw_lds[e] = v[u];
        }
    }
};


// Product of the scaling factors of the leading axes of image row r
// (row-major over axes 0..d-2), 32-bit index arithmetic.
__device__ __forceinline__ float row_scale(int d, const int *Nax, const float *const *scale, int r) {
    float sc = 1.0f;
    for (int a = d - 2; a >= 0; --a) {
        const int i = r % Nax[a];
        r /= Nax[a];
        sc *= scale[a][i];
    }
    return sc;
}

// row_scale with its loads issued at load() and the product formed at value(),
// so the loads overlap other work.
struct RowScale {
    float f[kMaxDim - 1];
    int n;
    __device__ __forceinline__ void load(int d, const int *Nax, const float *const *scale, int r) {
        n = d - 1;
#pragma unroll
        for (int a = kMaxDim - 2; a >= 0; --a) {
            if (a < n) {
                const int i = r % Nax[a];
                r /= Nax[a];
                f[a] = scale[a][i];
            }
        }
    }
    __device__ __forceinline__ float value() const {
        float sc = 1.0f;
#pragma unroll
        for (int a = kMaxDim - 2; a >= 0; --a)
            if (a < n) sc *= f[a];
        return sc;
    }
};

// Grid position of image index i on an axis of image size N and grid size K
// (n = i - N/2 wrapped modulo K), and its inverse (-1 in the zero gap).
__device__ __forceinline__ int pad_pos(int i, int N, int K) { return i < N / 2 ? K - N / 2 + i : i - N / 2; }
__device__ __forceinline__ int src_row(int q, int N, int K) {
    if (q < N / 2) return q + N / 2;
    if (q >= K - N / 2) return q - (K - N / 2);
    return -1;
}

// ------------------------------------------------------------ FFT kernels
// Dynamic LDS layout of every FFT kernel: [K twiddles][tile].
template <int THREADS>
__device__ __forceinline__ void first_pass_body(const FirstPassArgs &a, int lines_per_wg, int64_t bx) {
    extern __shared__ float2 lds[];
    const int K = a.K, N = a.N;
    float2 *tw = lds;
    float2 *s = lds + K;
    const int64_t total = int64_t(a.B) * a.C * a.rows;
    const int64_t l0 = bx * lines_per_wg;
    const int nl = int(min(int64_t(lines_per_wg), total - l0));  // 1..64
    // Line `lane` of the workgroup, known to that lane of every wavefront: the
    // image and coil row offsets and the product of the leading axes' scaling
    // factors (applied after the FFT, which is linear along the line).
    const int lane = threadIdx.x & 63;
    int xb = 0, cb = 0;
    RowScale rsf;
    {
        const int64_t l = l0 + min(lane, nl - 1);
        const int g = int(l / a.rows);
        const int r = int(l - int64_t(g) * a.rows);
        const int b = g / a.C;
        const int c = g - b * a.C;
        rsf.load(a.d, a.Nax, a.scale, r);  // consumed after the FFT
        xb = (b * int(a.rows) + r) * N;
        cb = (c * int(a.rows) + r) * N;
    }
    TwiddleStage<THREADS> tws;
    tws.load(a.tw, K);
    // the tile holds nl * K <= THREADS * kEPT elements: every load is issued
    // before the first use
    const int ne = nl * K;
    const FastDiv byK(K);
    const float *slast = a.scale[a.d - 1];
    // (loads land in registers without a default value, so no copy waits for
    // them; `live` marks the elements that read the image)
    // (branch-free: indices are clamped into the row and `live` marks the
    // elements that really read the image, so no load waits on another)
    float2 xv[kEPT], cv[kEPT];
    float sv[kEPT];
    unsigned live = 0;
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = min(int(threadIdx.x) + u * THREADS, ne - 1);
        const int lw = byK.div(e);
        const int i = src_row(byK.rem(e, lw), N, K);
        live |= (int(threadIdx.x) + u * THREADS < ne && i >= 0) ? 1u << u : 0u;
        const int ic = max(i, 0);
        // one grid per image row without coils: line l reads image row l
        const int xbl = a.C == 1 ? int(l0 + lw) * N : __shfl(xb, lw);
        xv[u] = a.x[xbl + ic];
        sv[u] = slast[ic];
        if (a.coils) cv[u] = a.coils[__shfl(cb, lw) + ic];
    }
    // values first, without branches (one wait for all loads), then the writes
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        float2 v = cscale(xv[u], sv[u]);
        if (a.coils) v = cmul(v, cv[u]);
        xv[u] = (live & (1u << u)) ? v : make_float2(0.f, 0.f);
    }
    tws.store(tw, K);
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = threadIdx.x + u * THREADS;
        if (e < ne) s[e] = xv[u];
    }
    __syncthreads();
    lds_fft<THREADS, false, false>(s, nl, K, K, 1, a.rp, tw);
    const float rs = rsf.value();
    float2 *out = a.out + l0 * K;
    float2 pv[kEPT], mv[kEPT];
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = min(int(threadIdx.x) + u * THREADS, ne - 1);
        const int lw = byK.div(e);
        const int q = byK.rem(e, lw);
        if (a.phase) pv[u] = a.phase[q];
        if (a.mult) mv[u] = a.mult[((l0 + lw) % a.rows) * K + q];
    }
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = min(int(threadIdx.x) + u * THREADS, ne - 1);
        float2 v = s[e];
        if (a.d > 1) v = cscale(v, __shfl(rs, byK.div(e)));  // row scale of the element's line
        if (a.phase) v = cmul(v, pv[u]);
        if (a.mult) v = cmul(v, mv[u]);
        pv[u] = v;
    }
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = threadIdx.x + u * THREADS;
        if (e < ne) out[e] = pv[u];
    }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_first_pass(FirstPassArgs a, int lines_per_wg) {
    first_pass_body<THREADS>(a, lines_per_wg, blockIdx.x);
}

// Many problems in one launch: workgroup b runs block blocks[b].y of problem
// blocks[b].x, whose arguments sit in jobs[blocks[b].x].
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_first_pass_multi(const FirstJob *__restrict__ jobs,
                                                             const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const FirstJob &j = jobs[b.x];
    first_pass_body<THREADS>(j.a, j.lpw, b.y);
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

// SPLIT (inverse only): the first inverse pass of an adjoint whose split
// gridding tiles are still partial tiles (its own instantiation, so the
// common passes keep their register budget).
template <int THREADS, bool INV, bool SPLIT>
__device__ __forceinline__ void strided_pass_body(const StridedPassArgs &a, int W, int64_t ntc, int64_t bid) {
    extern __shared__ float2 lds[];
    const int K = a.K;
    float2 *tw = lds;
    float2 *s = lds + K;
    const int64_t ct = bid % ntc;
    const int64_t rest = bid / ntc;
    const int64_t o = rest % a.outer;
    const int64_t g = rest / a.outer;
    const int64_t c0 = ct * W;
    const int wv = int(min(int64_t(W), a.inner - c0));
    const float2 *in = a.in + ((g * a.outer + o) * a.Lin) * a.inner + c0;
    float2 *out = a.out + ((g * a.outer + o) * a.Lout) * a.inner + c0;
    TwiddleStage<THREADS> tws;
    tws.load(a.tw, K);
    // the tile holds K * W <= THREADS * kEPT elements
    const int ne = K * W;
    const FastDiv byW(W);
    // (no default values in the load registers, so no copy waits for a load;
    // `live` marks the elements that read the input)
    float2 v[kEPT], mv[kEPT], pv[kEPT];
    unsigned live = 0;
    if constexpr (!SPLIT) {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * THREADS;
            const int q = byW.div(min(e, ne - 1));
            const int w = e - __umul24(q, W);
            // forward: grid row q takes image row src_row (zero rows when Lin < K,
            // the centring shift when Lin == K); inverse: the input is the grid
            const int i = INV ? q : src_row(q, a.Lin, K);
            if (e < ne && w < wv && i >= 0) {
                live |= 1u << u;
                v[u] = in[int64_t(i) * a.inner + w];
                if (a.mult) mv[u] = a.mult[(o * a.Lin + i) * a.inner + c0 + w];
                if (INV && a.phase) pv[u] = a.phase[q];
            }
        }
    } else {
        // First inverse pass of the adjoint: a cell of a split gridding tile is
        // the sum of its partial tiles in chunk order (the order, hence the bits,
        // of k_reduce_partials).  Grid row q on axis 0, column c0 + w over the
        // remaining axes; the input and the cell's split entry are loaded
        // together, the partial tiles after that.
        const FastDiv byT0(a.T[0]), byT1(a.T[1]), byT2(a.d > 2 ? a.T[2] : 1), byK2(a.d > 2 ? a.Kax[2] : 1);
        int2 sp[kEPT];
        int cellv[kEPT];
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = min(int(threadIdx.x) + u * THREADS, ne - 1);
            const int q = byW.div(e);
            const int w = min(e - __umul24(q, W), wv - 1);
            const int i = INV ? q : max(src_row(q, a.Lin, K), 0);
            live |= (int(threadIdx.x) + u * THREADS < ne && e - __umul24(q, W) < wv &&
                     (INV || src_row(q, a.Lin, K) >= 0)) ? 1u << u : 0u;
            // grid coordinates of the cell: k0 = q, then the column's axes
            const int c = int(c0) + w;
            int k1 = c, k2 = 0;
            if (a.d > 2) {
                k1 = byK2.div(c);
                k2 = byK2.rem(c, k1);
            }
            const int t0 = byT0.div(q), t1 = byT1.div(k1);
            int tile = t0 * a.nt[1] + t1;
            int cell = byT0.rem(q, t0) * a.T[1] + byT1.rem(k1, t1);
            if (a.d > 2) {
                const int t2 = byT2.div(k2);
                tile = tile * a.nt[2] + t2;
                cell = cell * a.T[2] + byT2.rem(k2, t2);
            }
            v[u] = in[int64_t(i) * a.inner + w];
            sp[u] = a.split_of_tile[tile];
            cellv[u] = cell;
            if (INV && a.phase) pv[u] = a.phase[q];  // (never with a Toeplitz product)
        }
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int n = sp[u].y;
            if (n > 0) {
                const float2 *pp = a.partials + (g * a.n_slots + sp[u].x) * a.tile_cells + cellv[u];
                // kReduceLanes interleaved sums (chunk c into sum c mod
                // kReduceLanes, in chunk order), then added in lane order
                float2 acc[kReduceLanes];
#pragma unroll
                for (int j = 0; j < kReduceLanes; ++j) acc[j] = make_float2(0.f, 0.f);
                for (int k0 = 0; k0 < n; k0 += kReduceLanes) {
                    float2 t[kReduceLanes];
#pragma unroll
                    for (int j = 0; j < kReduceLanes; ++j)
                        if (k0 + j < n) t[j] = pp[int64_t(k0 + j) * a.tile_cells];
#pragma unroll
                    for (int j = 0; j < kReduceLanes; ++j)
                        if (k0 + j < n) acc[j] = cadd(acc[j], t[j]);
                }
#pragma unroll
                for (int j = 1; j < kReduceLanes; ++j) acc[0] = cadd(acc[0], acc[j]);
                v[u] = acc[0];
            }
        }
    }
    // values first, without branches (one wait for all loads), then the writes
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        float2 x = v[u];
        if (!SPLIT && a.mult) x = cmul(x, mv[u]);
        if (INV && a.phase) x = cmulcj(pv[u], x);
        v[u] = (live & (1u << u)) ? x : make_float2(0.f, 0.f);
    }
    tws.store(tw, K);
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = threadIdx.x + u * THREADS;
        if (e < ne) s[e] = v[u];
    }
    __syncthreads();
    lds_fft<THREADS, INV, true>(s, W, K, 1, W, a.rp, tw);
    // Lout * W <= K * W outputs
    const int no = a.Lout * W;
    if (!INV && a.phase) {
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = min(int(threadIdx.x) + u * THREADS, no - 1);
            pv[u] = a.phase[byW.div(e)];
        }
    }
    // values first, without branches, then the writes
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = min(int(threadIdx.x) + u * THREADS, no - 1);
        const int i = byW.div(e);
        const int q = INV ? pad_pos(i, a.Lout, K) : i;
        float2 x = s[__umul24(q, W) + byW.rem(e, i)];
        if (!INV && a.phase) x = cmul(x, pv[u]);
        v[u] = x;
    }
#pragma unroll
    for (int u = 0; u < kEPT; ++u) {
        const int e = threadIdx.x + u * THREADS;
        const int i = byW.div(min(e, no - 1));
        const int w = e - __umul24(i, W);
        if (e < no && w < wv) out[int64_t(i) * a.inner + w] = v[u];
    }
}

template <int THREADS, bool INV, bool SPLIT>
__global__ __launch_bounds__(THREADS) void k_strided_pass(StridedPassArgs a, int W, int64_t ntc) {
    strided_pass_body<THREADS, INV, SPLIT>(a, W, ntc, xcd_block(blockIdx.x, gridDim.x));
}

template <int THREADS, bool INV, bool SPLIT>
__global__ __launch_bounds__(THREADS) void k_strided_pass_multi(const StridedJob *__restrict__ jobs,
                                                               const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const StridedJob &j = jobs[b.x];
    strided_pass_body<THREADS, INV, SPLIT>(j.a, j.W, j.ntc, b.y);
}

template <int THREADS>
__device__ __forceinline__ void last_pass_body(const LastPassArgs &a, int rows_per_wg, int coils_per_round, int64_t bx) {
    extern __shared__ float2 lds[];
    __shared__ float rsc[kMaxLinesPerWg];
    const int K = a.K, N = a.N, C = a.C;
    float2 *tw = lds;
    float2 *s = lds + K;
    const int64_t nrt = (a.rows + rows_per_wg - 1) / rows_per_wg;
    const int64_t b = bx / nrt;
    const int64_t r0 = (bx % nrt) * rows_per_wg;
    const int nr = int(min(int64_t(rows_per_wg), a.rows - r0));
    TwiddleStage<THREADS> tws;
    tws.load(a.tw, K);
    const float *slast = a.scale[a.d - 1];
    if (coils_per_round >= C) {
        const FastDiv byK(K), byN(N), byC(C);
        // all coils of the rows in one tile (nr * C * K <= THREADS * kEPT
        // elements, nr * N outputs): every load is issued before the first use.
        // Lane rr (< nr <= 64) of every wavefront holds row rr's scaling factor.
        RowScale rsf;
        rsf.load(a.d, a.Nax, a.scale, int(r0) + min(int(threadIdx.x & 63), nr - 1));
        const int nl = nr * C;
        const int ne = nl * K;
        float2 v[kEPT], pv[kEPT];
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = min(int(threadIdx.x) + u * THREADS, ne - 1);  // (clamped: every load is in bounds)
            const int lw = byK.div(e);
            const int q = byK.rem(e, lw);
            const int rr = byC.div(lw), cc = byC.rem(lw, rr);
            v[u] = a.in[((b * C + cc) * a.rows + r0 + rr) * K + q];
            if (a.phase) pv[u] = a.phase[q];
        }
        if (a.phase) {
#pragma unroll
            for (int u = 0; u < kEPT; ++u) v[u] = cmulcj(pv[u], v[u]);
        }
        tws.store(tw, K);
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * THREADS;
            if (e < ne) s[e] = v[u];
        }
        __syncthreads();
        lds_fft<THREADS, true, false>(s, nl, K, K, 1, a.rp, tw);
        const float rs = rsf.value();
        const int no = nr * N;
        float sv[kEPT];
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = min(int(threadIdx.x) + u * THREADS, no - 1);
            sv[u] = slast[byN.rem(e, byN.div(e))];
        }
        // values first (one wait for the scaling-factor loads), then the writes
        float2 res[kEPT];
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = min(int(threadIdx.x) + u * THREADS, no - 1);
            const int rr = byN.div(e), i = byN.rem(e, rr);
            const int q = pad_pos(i, N, K);
            float2 sum = make_float2(0.f, 0.f);
            if (a.coils) {
#pragma unroll 1
                for (int cc = 0; cc < C; ++cc)
                    sum = cadd(sum, cmulcj(a.coils[(int64_t(cc) * a.rows + r0 + rr) * N + i], s[(rr * C + cc) * K + q]));
            } else {
#pragma unroll 1
                for (int cc = 0; cc < C; ++cc) sum = cadd(sum, s[(rr * C + cc) * K + q]);
            }
            res[u] = cscale(sum, __shfl(rs, rr) * sv[u]);
        }
#pragma unroll
        for (int u = 0; u < kEPT; ++u) {
            const int e = threadIdx.x + u * THREADS;
            const int rr = byN.div(min(e, no - 1)), i = e - __umul24(rr, N);
            if (e < no) a.x[(b * a.rows + r0 + rr) * N + i] = res[u];
        }
        return;
    }
    // more coils than one tile holds (C * K > the tile): rounds of
    // coils_per_round coils summed in LDS accumulators after the tile
    tws.store(tw, K);
    if (threadIdx.x < nr) rsc[threadIdx.x] = row_scale(a.d, a.Nax, a.scale, int(r0) + threadIdx.x);
    float2 *acc = s + rows_per_wg * coils_per_round * K;
    for (int e = threadIdx.x; e < nr * N; e += THREADS) acc[e] = make_float2(0.f, 0.f);
    for (int c0 = 0; c0 < C; c0 += coils_per_round) {
        const int nc = min(coils_per_round, C - c0);
        const int nl = nr * nc;
        for (int e = threadIdx.x; e < nl * K; e += THREADS) {
            const int lw = e / K, q = e - lw * K;
            const int rr = lw / nc, cc = lw - rr * nc;
            float2 v = a.in[((b * C + c0 + cc) * a.rows + r0 + rr) * K + q];
            if (a.phase) v = cmulcj(a.phase[q], v);
            s[e] = v;
        }
        __syncthreads();
        lds_fft<THREADS, true, false>(s, nl, K, K, 1, a.rp, tw);
        for (int e = threadIdx.x; e < nr * N; e += THREADS) {
            const int rr = e / N, i = e - rr * N;
            const int q = pad_pos(i, N, K);
            float2 sum = make_float2(0.f, 0.f);
            for (int cc = 0; cc < nc; ++cc) {
                float2 t = s[(rr * nc + cc) * K + q];
                if (a.coils) t = cmulcj(a.coils[(int64_t(c0 + cc) * a.rows + r0 + rr) * N + i], t);
                sum = cadd(sum, t);
            }
            acc[e] = cadd(acc[e], sum);
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < nr * N; e += THREADS) {
        const int rr = e / N, i = e - rr * N;
        a.x[(b * a.rows + r0 + rr) * N + i] = cscale(acc[e], rsc[rr] * slast[i]);
    }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_last_pass(LastPassArgs a, int rows_per_wg, int coils_per_round) {
    last_pass_body<THREADS>(a, rows_per_wg, coils_per_round, blockIdx.x);
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_last_pass_multi(const LastJob *__restrict__ jobs,
                                                            const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    const LastJob &j = jobs[b.x];
    last_pass_body<THREADS>(j.a, j.rpw, j.cpr, b.y);
}

// FFT tile sizes: a tile holds up to THREADS * kEPT elements.  The host takes
// the largest tile that still leaves about target_groups workgroups (small
// transforms spread over the whole chip), then the smallest block that holds
// it.

template <template <int> class L, class A>
hipError_t fft_dispatch(int threads, const A &a, hipStream_t s, int p0, int64_t p1, size_t lds, unsigned blocks) {
    switch (threads) {
        case 64: return L<64>::go(a, s, p0, p1, lds, blocks);
        case 128: return L<128>::go(a, s, p0, p1, lds, blocks);
        case 256: return L<256>::go(a, s, p0, p1, lds, blocks);
        default: return L<512>::go(a, s, p0, p1, lds, blocks);
    }
}

int threads_for(int elems) {
    int t = 64;
    while (t < 512 && t * kEPT < elems) t *= 2;
    return t;
}

template <int T>
struct FirstGo {
    static hipError_t go(const FirstPassArgs &a, hipStream_t s, int lpw, int64_t, size_t lds, unsigned blocks) {
        launch_kernel(k_first_pass<T>, dim3(blocks), dim3(T), lds, s, a, lpw);
        return hipGetLastError();
    }
};

template <int T>
struct StridedGoF {
    static hipError_t go(const StridedPassArgs &a, hipStream_t s, int W, int64_t ntc, size_t lds, unsigned blocks) {
        launch_kernel((k_strided_pass<T, false, false>), dim3(blocks), dim3(T), lds, s, a, W, ntc);
        return hipGetLastError();
    }
};

template <int T>
struct StridedGoI {
    static hipError_t go(const StridedPassArgs &a, hipStream_t s, int W, int64_t ntc, size_t lds, unsigned blocks) {
        if (a.split_of_tile)
            launch_kernel((k_strided_pass<T, true, true>), dim3(blocks), dim3(T), lds, s, a, W, ntc);
        else
            launch_kernel((k_strided_pass<T, true, false>), dim3(blocks), dim3(T), lds, s, a, W, ntc);
        return hipGetLastError();
    }
};

}  // namespace

// ------------------------------------------------------------ launchers
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
    L.lds = size_t(lpw + 1) * a.K * sizeof(float2);
    L.p0 = lpw;
    return L;
}

hipError_t launch_first_pass(const FirstPassArgs &a, hipStream_t s) {
    const FftLaunch L = first_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    return fft_dispatch<FirstGo>(L.threads, a, s, L.p0, 0, L.lds, unsigned(L.blocks));
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
    L.lds = size_t(W + 1) * a.K * sizeof(float2);
    L.p0 = int(W);
    L.p1 = ntc;
    return L;
}

hipError_t launch_strided_pass(const StridedPassArgs &a, hipStream_t s) {
    const FftLaunch L = strided_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    if (a.inverse) return fft_dispatch<StridedGoI>(L.threads, a, s, L.p0, L.p1, L.lds, unsigned(L.blocks));
    return fft_dispatch<StridedGoF>(L.threads, a, s, L.p0, L.p1, L.lds, unsigned(L.blocks));
}

namespace {
template <int T>
struct LastGo {
    static hipError_t go(const LastPassArgs &a, hipStream_t s, int rpw, int64_t cpr, size_t lds, unsigned blocks) {
        launch_kernel(k_last_pass<T>, dim3(blocks), dim3(T), lds, s, a, rpw, int(cpr));
        return hipGetLastError();
    }
};
}  // namespace

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
    const bool one_round = coils_per_round >= a.C;
    L.lds = (size_t(a.K) + size_t(rows_per_wg) * coils_per_round * a.K +
             (one_round ? 0 : size_t(rows_per_wg) * a.N)) * sizeof(float2);
    L.p0 = rows_per_wg;
    L.p1 = coils_per_round;
    return L;
}

hipError_t launch_last_pass(const LastPassArgs &a, hipStream_t s) {
    const FftLaunch L = last_pass_launch(a);
    if (L.blocks == 0) return hipSuccess;
    return fft_dispatch<LastGo>(L.threads, a, s, L.p0, L.p1, L.lds, unsigned(L.blocks));
}

// ---- many problems per launch
namespace {
template <int T>
struct FirstMulti {
    static void go(const FirstJob *j, const int4 *b, int64_t n, size_t lds, hipStream_t s) {
        launch_kernel(k_first_pass_multi<T>, dim3(unsigned(n)), dim3(T), lds, s, j, b);
    }
};
template <int T>
struct LastMulti {
    static void go(const LastJob *j, const int4 *b, int64_t n, size_t lds, hipStream_t s) {
        launch_kernel(k_last_pass_multi<T>, dim3(unsigned(n)), dim3(T), lds, s, j, b);
    }
};
template <bool INV, bool SPLIT>
struct StridedMultiF {
    template <int T>
    struct K {
        static void go(const StridedJob *j, const int4 *b, int64_t n, size_t lds, hipStream_t s) {
            launch_kernel((k_strided_pass_multi<T, INV, SPLIT>), dim3(unsigned(n)), dim3(T), lds, s, j, b);
        }
    };
};

template <template <int> class L, class Job>
hipError_t threads_go(int threads, const Job *j, const int4 *b, int64_t n, size_t lds, hipStream_t s) {
    if (n == 0) return hipSuccess;
    switch (threads) {
        case 64: L<64>::go(j, b, n, lds, s); break;
        case 128: L<128>::go(j, b, n, lds, s); break;
        case 256: L<256>::go(j, b, n, lds, s); break;
        case 512: L<512>::go(j, b, n, lds, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_first_pass_multi(const FirstJob *jobs, const int4 *blocks, int64_t nblocks, int threads,
                                   size_t lds, hipStream_t s) {
    return threads_go<FirstMulti>(threads, jobs, blocks, nblocks, lds, s);
}

hipError_t launch_strided_pass_multi(const StridedJob *jobs, const int4 *blocks, int64_t nblocks, int threads,
                                     bool inverse, bool split, size_t lds, hipStream_t s) {
    if (!inverse) return threads_go<StridedMultiF<false, false>::K>(threads, jobs, blocks, nblocks, lds, s);
    if (split) return threads_go<StridedMultiF<true, true>::K>(threads, jobs, blocks, nblocks, lds, s);
    return threads_go<StridedMultiF<true, false>::K>(threads, jobs, blocks, nblocks, lds, s);
}

hipError_t launch_last_pass_multi(const LastJob *jobs, const int4 *blocks, int64_t nblocks, int threads, size_t lds,
                                  hipStream_t s) {
    return threads_go<LastMulti>(threads, jobs, blocks, nblocks, lds, s);
}

}  // namespace nufft
