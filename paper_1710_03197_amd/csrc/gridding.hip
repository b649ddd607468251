// Gridding V^H (paper Section 2.1 "Adjoint PyNUFFT"):
//   k_grid_blk     in 3D on the matrix cores by 4 x 4 blocks;
//   k_grid_cols    in 2D for several grids, by 4 x 4 blocks with the grids as
//                  columns;
//   k_grid_mfma    by row tiles (2D and other 16-cell tiles);
//   k_grid         on the vector ALUs (other tiles).  All output driven: a
//                  work item owns one grid tile and walks the samples that
//                  reach it (staged in LDS), so the tile is written once with
//                  plain stores: no memset, no atomics, a fixed summation
//                  order; crowded tiles are split into chunks whose partial
//                  tiles k_reduce_partials (or the first inverse FFT pass)
//                  sums in a fixed order.
// All arithmetic is float32 with float32 accumulation; window positions are
// float64 (u = omega * K/(2 pi) as one rounded multiply).
#include "device.h"

namespace nufft {
namespace {

// ------------------------------------------------------------ work distribution
// Work items (gather chunks, gridding tile chunks) are ordered by decreasing
// size on the host; workgroup b runs item b, and the hardware deals
// consecutive workgroups round-robin over the 8 XCDs, so the heavy items
// spread over the whole chip.

// ------------------------------------------------------------ V^H (output-driven gridding)
// One workgroup per (tile, chunk).  The samples that reach the tile are the
// tile's own bin plus, from each lower neighbour bin, only the sub-bins whose
// windows cross into this tile (tile_segments).
//
// No atomics: the tile's rows (leading coordinates) are cut into segments of
// LS cells along the last axis, one segment per lane, held in registers.
// Samples are staged in LDS in batches: window offsets along the leading
// axes, their per-axis weights, the value, and the last-axis weights already
// expanded into a zero-padded row of the tile (so the inner loop needs no
// tap index and no branch).  Every lane of a group then walks the group's
// batch and adds LS weighted values per sample.  Lane groups split the
// samples; their register tiles are summed through LDS at the end in group
// order, so the result does not depend on scheduling.
constexpr int kGridThreads = 256;

// Synchronise a lane group's LDS traffic: a single wavefront only needs its
// own LDS operations ordered (lockstep execution), larger groups need the
// workgroup barrier.
__device__ __forceinline__ void group_sync(int gsize) {
    if (gsize == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// The sorted-sample segments that reach the work item's tile (its own bin and
// the crossing sub-bins of its lower neighbours, in tile_segments order), from
// the item's table made when the plan was built: segment starts into seg_lo,
// their offsets in the item's sample list (and the total) into seg_pre.  Needs
// nothing from the item record, so both loads are in flight together.  Every
// thread of the workgroup calls it; returns the number of segments.
__device__ __forceinline__ int grid_item_segments(const GridArgs &a, int64_t item, int *seg_lo, int *seg_pre) {
    if (threadIdx.x <= a.n_kinds) {
        const int2 e = a.item_segs[item * (a.n_kinds + 1) + threadIdx.x];
        seg_lo[threadIdx.x] = e.x;
        seg_pre[threadIdx.x] = e.y;
    }
    __syncthreads();
    return a.n_kinds;
}

// Segment of item sample f (the last segment whose start is <= f) for a batch
// of consecutive samples fb .. fb + span - 1.  `cursor` is uniform over the
// batch's lanes and kept across the item's batches, which only move forward:
// it is advanced to the batch's first sample, then every segment start inside
// the batch adds one for the lanes at or past it.  The same segment as a scan
// from segment 0, without a divergent per-lane loop.
__device__ __forceinline__ int batch_segment(const int *seg_pre, int nseg, int &cursor, int fb, int span, int f) {
    while (cursor + 1 < nseg && seg_pre[cursor + 1] <= fb) ++cursor;
    int sg = cursor;
    for (int k = cursor + 1; k < nseg && seg_pre[k] < fb + span; ++k) sg += seg_pre[k] <= f ? 1 : 0;
    return sg;
}

template <int DIM, int LS, int JP>
__device__ __forceinline__ void grid_body(const GridArgs &a, int64_t item, int g) {
    extern __shared__ float4 stage_mem[];  // float4: 16-byte aligned rows for the vector reads
    float *stage = reinterpret_cast<float *>(stage_mem);
    __shared__ int seg_lo[kMaxNeighbors + 1];
    __shared__ int seg_pre[kMaxNeighbors + 1];
    const GridItem it = a.items[item];
    const int nseg = grid_item_segments(a, item, seg_lo, seg_pre);
    const int J = a.geo.J;
    const int L = a.T[DIM - 1];           // cells per tile row
    const int S = a.segs;                 // segments per row
    const int Lp = S * LS;                // padded row length
    const int lead = a.tile_cells / L;    // rows of the tile
    const int gsize = a.group_lanes;      // lanes per sample group (multiple of 64, >= lead * S)
    const int ngroups = kGridThreads / gsize;
    const int grp = threadIdx.x / gsize;
    const int lane = threadIdx.x - grp * gsize;
    const int B = gsize;                  // samples per batch and group
    const int BP = B + 1;
    // staged arrays of this group
    float *gbase = stage + grp * a.stage_floats;
    float *wrow = gbase;                              // [B][Lp] last-axis weights on the row
    float *sv = wrow + B * Lp;                        // [2][BP] value
    int *so = reinterpret_cast<int *>(sv + 2 * BP);   // [DIM-1][BP] leading first-tap offsets
    float *sw = sv + 2 * BP + (DIM - 1) * BP;         // [DIM-1][J][BP] leading weights

    int tc[DIM];
    {
        int t = it.tile;
#pragma unroll
        for (int ax = DIM - 1; ax >= 0; --ax) {
            tc[ax] = t % a.nt[ax];
            t /= a.nt[ax];
        }
    }
    const int total = seg_pre[nseg];
    const int f0 = it.chunk * a.chunk;
    const int n = min(total, f0 + a.chunk) - f0;
    int base[DIM];
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) base[ax] = tc[ax] * a.T[ax];
    // this lane's segment: row (leading coordinates) and first cell
    const int row = lane / S;
    const int cseg = (lane - row * S) * LS;
    int lc[DIM];
    {
        int r = row;
#pragma unroll
        for (int ax = DIM - 2; ax >= 0; --ax) {
            lc[ax] = r % a.T[ax];
            r /= a.T[ax];
        }
        lc[DIM - 1] = cseg;
    }
    const bool row_ok = row < lead;
    const float2 *y = a.y + int64_t(g) * a.M;
    float2 acc[LS];
#pragma unroll
    for (int c = 0; c < LS; ++c) acc[c] = make_float2(0.f, 0.f);

    // A group of one wavefront stages and consumes its own batches, so it
    // synchronises only with itself and runs ahead of the other groups.
    const int per_iter = B * ngroups;
    int cursor = 0;
    for (int b0 = 0; b0 < n; b0 += per_iter) {
        // ---- stage one batch per group: lane `lane` stages sample b0 + grp*B + lane
        const int s_idx = b0 + grp * B + lane;
        const int sg = batch_segment(seg_pre, nseg, cursor, f0 + b0 + grp * B, B, f0 + s_idx);
        if (s_idx < n) {
            const int f = f0 + s_idx;
            const int64_t i = seg_lo[sg] + (f - seg_pre[sg]);
            float wl_row[JP];  // last-axis weights, spread on the row below
            int o_last = 0;
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) {
                const double u = __dmul_rn(double(a.om_sorted[i * DIM + ax]), a.geo.C[ax]);
                // (min-max: taps wrapping past K carry a sign, see mm_phase)
                const double k0 = floor(u - 0.5 * J) + 1.0;
                const float fr = float(u - k0 - (0.5 * J - 1.0));
                const int K = a.geo.K[ax];
                const int kw = wrap_first_tap(k0, K);
                int o = kw - base[ax];
                if (a.nt[ax] > 1 && o >= a.T[ax]) o -= K;  // window wrapping in from the top
                const float z = 2.0f * fr - 1.0f;
                float wv[JP];
                poly_rows<JP>(a.geo.coef[ax], JP, a.geo.nq[ax], z, wv);
                if (a.geo.minmax) mm_sign_taps<JP>(wv, K - int(kw));
#pragma unroll
                for (int j = 0; j < JP; ++j) {
                    if (j < J) {
                        if (ax < DIM - 1)
                            sw[(ax * J + j) * BP + lane] = wv[j];
                        else
                            wl_row[j] = wv[j];
                    }
                }
                if (ax < DIM - 1) so[ax * BP + lane] = o;
                else o_last = o;
            }
            // the tile row of last-axis weights: cell c gets w[c - o] (wrapping
            // when the axis is one tile), built in registers and stored with
            // 16-byte writes
            const int Kl = a.geo.K[DIM - 1];
            const bool wrapl = a.nt[DIM - 1] == 1;
            float4 *wr4 = reinterpret_cast<float4 *>(wrow + lane * Lp);
            for (int c4 = 0; c4 < Lp; c4 += 4) {
                float r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    int j = c4 + u - o_last;
                    if (wrapl && j < 0) j += Kl;
                    float v = 0.f;
#pragma unroll
                    for (int jj = 0; jj < JP; ++jj)
                        if (jj < J && j == jj) v = wl_row[jj];
                    r[u] = (c4 + u < L) ? v : 0.f;
                }
                wr4[c4 >> 2] = make_float4(r[0], r[1], r[2], r[3]);
            }
            float2 v = a.y_sorted ? y[i] : y[a.perm[i]];
            if (a.geo.minmax) v = cmulcj(mm_phase<DIM>(a.geo, a.om_sorted + i * DIM), v);
            sv[lane] = v.x;
            sv[BP + lane] = v.y;
        }
        group_sync(gsize);
        // ---- every lane of the group walks the group's batch
        const int nb = min(B, n - (b0 + grp * B));
#pragma unroll 2
        for (int s = 0; s < nb; ++s) {
            float wl = row_ok ? 1.f : 0.f;
#pragma unroll
            for (int ax = 0; ax < DIM - 1; ++ax) {
                int j = lc[ax] - so[ax * BP + s];
                if (a.nt[ax] == 1 && j < 0) j += a.geo.K[ax];
                const bool in = (j >= 0) && (j < J);
                const float w = sw[(ax * J + (in ? j : 0)) * BP + s];
                wl = in ? wl * w : 0.f;
            }
            const float vr = sv[s] * wl, vi = sv[BP + s] * wl;
            const float4 *wr4 = reinterpret_cast<const float4 *>(wrow + s * Lp + cseg);
#pragma unroll
            for (int q = 0; q < LS / 4; ++q) {
                const float4 w = wr4[q];
                acc[4 * q + 0].x = fmaf(w.x, vr, acc[4 * q + 0].x);
                acc[4 * q + 0].y = fmaf(w.x, vi, acc[4 * q + 0].y);
                acc[4 * q + 1].x = fmaf(w.y, vr, acc[4 * q + 1].x);
                acc[4 * q + 1].y = fmaf(w.y, vi, acc[4 * q + 1].y);
                acc[4 * q + 2].x = fmaf(w.z, vr, acc[4 * q + 2].x);
                acc[4 * q + 2].y = fmaf(w.z, vi, acc[4 * q + 2].y);
                acc[4 * q + 3].x = fmaf(w.w, vr, acc[4 * q + 3].x);
                acc[4 * q + 3].y = fmaf(w.w, vi, acc[4 * q + 3].y);
            }
        }
        group_sync(gsize);
    }
    // ---- combine the groups' register tiles (group order), write the tile
    float2 *red = reinterpret_cast<float2 *>(stage);  // [ngroups][lead][Lp], reuses the staging LDS
    const bool seg_ok = row_ok;
    if (ngroups > 1) {
        __syncthreads();  // every group is done with its staging area
        if (seg_ok) {
#pragma unroll
            for (int c = 0; c < LS; ++c) red[(grp * lead + row) * Lp + cseg + c] = acc[c];
        }
        __syncthreads();
    }
    const bool to_partial = it.nchunks > 1;
    float2 *dst = to_partial ? a.partials + (int64_t(g) * a.n_slots + it.slot + it.chunk) * a.tile_cells
                             : a.h + int64_t(g) * a.grid_elems;
    if (ngroups == 1) {
        if (seg_ok) {
            int64_t idx;
            if (to_partial) {
                idx = int64_t(row) * L + cseg;
            } else {
                idx = 0;
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) idx = idx * a.geo.K[ax] + base[ax] + lc[ax];
            }
#pragma unroll
            for (int c = 0; c < LS; ++c)
                if (cseg + c < L) dst[idx + c] = acc[c];
        }
    } else {
        for (int e = threadIdx.x; e < lead * L; e += kGridThreads) {
            const int r = e / L, c = e - r * L;
            float2 sum = red[r * Lp + c];
            for (int q = 1; q < ngroups; ++q) sum = cadd(sum, red[(q * lead + r) * Lp + c]);
            int64_t idx;
            if (to_partial) {
                idx = e;
            } else {
                int rr = r;
                int l[DIM];
                l[DIM - 1] = c;
#pragma unroll
                for (int ax = DIM - 2; ax >= 0; --ax) {
                    l[ax] = rr % a.T[ax];
                    rr /= a.T[ax];
                }
                idx = 0;
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) idx = idx * a.geo.K[ax] + base[ax] + l[ax];
            }
            dst[idx] = sum;
        }
    }
}

template <int DIM, int LS, int JP>
__global__ __launch_bounds__(kGridThreads) void k_grid(GridArgs a) {
    grid_body<DIM, LS, JP>(a, blockIdx.x, blockIdx.y);
}

template <int DIM, int LS, int JP>
__global__ __launch_bounds__(kGridThreads) void k_grid_multi(const GridArgs *__restrict__ jobs,
                                                            const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    grid_body<DIM, LS, JP>(jobs[b.x], b.y, b.z);
}

// V^H on the matrix cores, for tiles of 16*MB rows (the leading axes) by 16
// cells (last axis).  Over a batch of samples s the tile is
//   H[r][c] = sum_s (v_s * wlead_s[r]) * wlast_s[c],
// a product of a rows x samples matrix and a samples x 16 matrix, i.e.
// 16x16x4 fp32 MFMAs with the samples as the reduction dimension (real and
// imaginary parts as two products sharing the wlast operand).  Each wave
// stages 64 samples in LDS: the values of the GP grids the workgroup grids
// (coils or batch entries share the trajectory, so the window weights are
// staged once for all of them) and, per axis, the sample's weights spread
// over the tile's T_a coordinates (zero outside the window, window wrapping
// resolved here), so in the walk lane (i + 16k) reads A[i][k] and B[k][i] of
// sample k at fixed offsets.  The four waves take different samples of the
// item and their tiles are summed in LDS in wave order (deterministic).
typedef float mfma_f4 __attribute__((ext_vector_type(4)));

template <int DIM, int NJ, int MB, int GP, bool TAB>
__device__ __forceinline__ void grid_mfma_body(const GridArgs &a, int64_t item, int gg) {
    extern __shared__ float mf_lds[];
    __shared__ int seg_lo[kMaxNeighbors + 1];
    __shared__ int seg_pre[kMaxNeighbors + 1];
    const GridItem it = a.items[item];
    const int nseg = grid_item_segments(a, item, seg_lo, seg_pre);
    const int J = a.geo.J;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform per wavefront
    const int lane = threadIdx.x & 63;
    const int g0 = gg * GP;                        // first grid of this workgroup
    const int ng = min(GP, a.grids - g0);          // grids it writes
    int tsum = 0;
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) tsum += a.T[ax];
    const int RS = (2 * GP + tsum) | 1;  // floats per staged sample: GP values, then T_a weights per axis (odd)
    float *rec = mf_lds + wave * 64 * RS;

    int tc[DIM];
    {
        int t = it.tile;
#pragma unroll
        for (int ax = DIM - 1; ax >= 0; --ax) {
            tc[ax] = t % a.nt[ax];
            t /= a.nt[ax];
        }
    }
    const int total = seg_pre[nseg];
    const int f0 = it.chunk * a.chunk;
    const int n = min(total, f0 + a.chunk) - f0;
    int base[DIM], width[DIM], off[DIM];
    {
        int o = 2 * GP;
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) {
            base[ax] = tile_base(tc[ax], a.geo.K[ax], a.T[ax], a.nt[ax]);
            width[ax] = tile_base(tc[ax] + 1, a.geo.K[ax], a.T[ax], a.nt[ax]) - base[ax];
            off[ax] = o;
            o += a.T[ax];
        }
    }

    // this lane's record offsets: A operand (leading weights of row
    // 16 blk + rl, per row block) and B operand (last-axis weight of column rl)
    const int rl = lane & 15;
    const int kq = lane >> 4;
    int aoff[MB][DIM - 1];
#pragma unroll
    for (int blk = 0; blk < MB; ++blk) {
        int r = blk * 16 + rl;
#pragma unroll
        for (int ax = DIM - 2; ax >= 0; --ax) {
            aoff[blk][ax] = off[ax] + r % a.T[ax];
            r /= a.T[ax];
        }
    }
    const int boff = off[DIM - 1] + rl;
    mfma_f4 acc_re[GP][MB], acc_im[GP][MB];
#pragma unroll
    for (int q = 0; q < GP; ++q) {
#pragma unroll
        for (int blk = 0; blk < MB; ++blk) {
            acc_re[q][blk] = mfma_f4{0.f, 0.f, 0.f, 0.f};
            acc_im[q][blk] = mfma_f4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // The global reads of a batch (trajectory, sample values) are issued one
    // batch ahead, so they are in flight while the wave walks the current one.
    float pom[DIM];
    float4 prec[TAB ? table_f4(DIM, NJ) : 1];
    float2 pv[GP];
    bool pvalid = false;
    int cursor = 0;
    auto fetch = [&](int b) {
        const int s_idx = b + wave * 64 + lane;
        pvalid = s_idx < n;
        const int sg = batch_segment(seg_pre, nseg, cursor, f0 + b + wave * 64, 64, f0 + s_idx);
        if (pvalid) {
            const int f = f0 + s_idx;
            const int64_t i = seg_lo[sg] + (f - seg_pre[sg]);
            if constexpr (TAB) {
                load_window_record<NJ, DIM>(a.geo, i, prec);
            } else {
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) pom[ax] = a.om_sorted[i * DIM + ax];
            }
            const int64_t src = a.y_sorted ? i : int64_t(a.perm[i]);
#pragma unroll
            for (int q = 0; q < GP; ++q)
                pv[q] = q < ng ? a.y[int64_t(g0 + q) * a.M + src] : make_float2(0.f, 0.f);
        }
    };
    fetch(0);
    for (int b0 = 0; b0 < n; b0 += 256) {
        // ---- stage: lane = sample b0 + 64 * wave + lane of the item
        float *my = rec + lane * RS;
        {
            float2 ph = make_float2(1.f, 0.f);
            if constexpr (!TAB)
                if (pvalid && a.geo.minmax) ph = mm_phase<DIM>(a.geo, pom);
#pragma unroll
            for (int q = 0; q < GP; ++q) {
                const float2 v = pvalid ? (a.geo.minmax ? cmulcj(ph, pv[q]) : pv[q]) : make_float2(0.f, 0.f);
                my[2 * q] = v.x;
                my[2 * q + 1] = v.y;
            }
        }
        int kwa[DIM];
        float wva[DIM][NJ];
        if (pvalid) {
            if constexpr (TAB)
                unpack_window<NJ, DIM>(prec, kwa, wva);
            else
                eval_window<NJ, DIM>(a.geo, pom, kwa, wva);
        }
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) {
            float *E = my + off[ax];
            const int T = a.T[ax];
#pragma unroll 4
            for (int x = 0; x < T; ++x) E[x] = 0.f;
            if (pvalid) {
                const int K = a.geo.K[ax];
                const int kw = kwa[ax];
                const int o = kw - base[ax];  // first tap relative to the tile, in [-base, K - base)
                float *wv = wva[ax];
                if (a.geo.minmax) mm_sign_taps<NJ>(wv, K - kw);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (j < J) {
                        int x = o + j;
                        if (x >= K) x -= K;  // taps wrapping past the top of the axis
                        if (x >= 0 && x < T) E[x] = wv[j];
                    }
                }
            }
        }
        if (b0 + 256 < n) fetch(b0 + 256);
        group_sync(64);
        // ---- walk: 4 samples per step
        const int nb = min(64, n - (b0 + wave * 64));
#pragma unroll 2
        for (int st = 0; st * 4 < nb; ++st) {
            const float *sr = rec + (st * 4 + kq) * RS;
            float vx[GP], vy[GP];
#pragma unroll
            for (int q = 0; q < GP; ++q) {
                vx[q] = sr[2 * q];
                vy[q] = sr[2 * q + 1];
            }
            const float bw = sr[boff];
#pragma unroll
            for (int blk = 0; blk < MB; ++blk) {
                float wl = sr[aoff[blk][0]];
#pragma unroll
                for (int ax = 1; ax < DIM - 1; ++ax) wl *= sr[aoff[blk][ax]];
#pragma unroll
                for (int q = 0; q < GP; ++q) {
                    acc_re[q][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx[q] * wl, bw, acc_re[q][blk], 0, 0, 0);
                    acc_im[q][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(vy[q] * wl, bw, acc_im[q][blk], 0, 0, 0);
                }
            }
        }
        group_sync(64);
    }
    // ---- per grid: sum the waves' tiles in wave order and write the tile
    const int cells = MB * 256;
    float2 *red = reinterpret_cast<float2 *>(mf_lds);  // [4][cells], reuses the staging LDS
#pragma unroll
    for (int q = 0; q < GP; ++q) {
        __syncthreads();  // every wave is done with the staging area / the previous grid's sums
#pragma unroll
        for (int blk = 0; blk < MB; ++blk) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = blk * 16 + 4 * kq + r;  // D[row][col] sits in lane col + 16 (row / 4), register row % 4
                red[wave * cells + row * 16 + rl] = make_float2(acc_re[q][blk][r], acc_im[q][blk][r]);
            }
        }
        __syncthreads();
        if (q < ng) {
            const int g = g0 + q;
            const bool to_partial = it.nchunks > 1;
            float2 *dst = to_partial ? a.partials + (int64_t(g) * a.n_slots + it.slot + it.chunk) * a.tile_cells
                                     : a.h + int64_t(g) * a.grid_elems;
            for (int e = threadIdx.x; e < cells; e += 256) {
                float2 sum = red[e];
#pragma unroll
                for (int w = 1; w < 4; ++w) sum = cadd(sum, red[w * cells + e]);
                int64_t idx;
                if (to_partial) {
                    idx = e;
                } else {
                    int rr = e >> 4;
                    int l[DIM];
                    l[DIM - 1] = e & 15;
#pragma unroll
                    for (int ax = DIM - 2; ax >= 0; --ax) {
                        l[ax] = rr % a.T[ax];
                        rr /= a.T[ax];
                    }
                    idx = 0;
                    bool in = true;
#pragma unroll
                    for (int ax = 0; ax < DIM; ++ax) {
                        idx = idx * a.geo.K[ax] + base[ax] + l[ax];
                        in = in && l[ax] < width[ax];
                    }
                    if (!in) continue;  // past the tile's own cells
                }
                dst[idx] = sum;
            }
        }
    }
}

template <int DIM, int NJ, int MB, int GP, bool TAB>
__global__ __launch_bounds__(256) void k_grid_mfma(GridArgs a) {
    grid_mfma_body<DIM, NJ, MB, GP, TAB>(a, blockIdx.x, blockIdx.y);
}

template <int DIM, int NJ, int MB, int GP, bool TAB>
__global__ __launch_bounds__(256) void k_grid_mfma_multi(const GridArgs *__restrict__ jobs,
                                                        const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    grid_mfma_body<DIM, NJ, MB, GP, TAB>(jobs[b.x], b.y, b.z);
}

// V^H on the matrix cores in 2D for several grids (coils, batch entries) that
// share the trajectory: 16 x 16 tiles, one or four wavefronts per work item and
// group of kColGrids grids.  The tile is cut into 4 x 4 blocks, and a block is one
// product over the samples whose columns are the grids' real and imaginary
// parts:
//   H[(x0, x1)][2 g + part] = sum_s (w0_s[x0] w1_s[x1]) v_{s,g,part}
// (v_mfma_f32_16x16x4_f32; eight grids fill its 16 columns).  A J = 6 window
// covers 36 of the 81 cells of the blocks it reaches on average, against 36 of
// 256 in the row-tile form, whose columns are cells, and a product serves eight
// grids.  Staging is the block kernel's: 64 samples per batch (weights spread
// over the tile, taps outside it to a discard slot, the set of blocks reached),
// then block by block the groups of four samples that reach it.  Bound by LDS
// latency and reads (four per two products) and the staging.  Measured, row-tile
// form -> this: 8 grids of 640 x 640, M = 128000: 72 -> 30 us; 24 grids of 256 x
// 256, M = 20011: 54 -> 28 us; 24 spirals x 8 coils: 1215 -> 450 us.
//
// A batch's products with a block are one chain from zero, and an item's chains
// are added in batch order.  NW = 1: one wavefront does all of it.  NW = 4: four
// wavefronts stage a batch each and then walk all four, each for its own row of
// blocks.  Both give the same bits, so a problem's result does not depend on what
// shares its launch, and chains of 64 samples round less than the one chain over
// all of a wavefront's batches that they replace (adjoint of 24 spirals x 8 coils
// against float64 1.13e-7 -> 1.02e-7; 1768 -> 1766 us a pass).
template <int NJ, bool TAB, int NW>
__device__ __forceinline__ void grid_cols_body(const GridArgs &a, int64_t item, int gg) {
    constexpr int T = 16, ROWS = 4 / NW;
    constexpr int RS = 2 * T + 1;            // weights of a sample, then the discard slot (odd)
    constexpr int VS = 2 * kColGrids + 1;    // its values (odd)
    extern __shared__ float col_lds[];
    __shared__ int seg_lo[kMaxNeighbors + 1];
    __shared__ int seg_pre[kMaxNeighbors + 1];
    const GridItem it = a.items[item];
    const int nseg = grid_item_segments(a, item, seg_lo, seg_pre);
    const int J = a.geo.J;
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    float *rec = col_lds;                                             // [NW][64][RS]
    float *val = rec + NW * 64 * RS;                           // [NW][64][VS]
    unsigned *smask = reinterpret_cast<unsigned *>(val + NW * 64 * VS);  // [NW][64]
    const int t0 = it.tile / a.nt[1];
    const int t1 = it.tile - t0 * a.nt[1];
    const int base[2] = {tile_base(t0, a.geo.K[0], T, a.nt[0]), tile_base(t1, a.geo.K[1], T, a.nt[1])};
    const int width[2] = {tile_base(t0 + 1, a.geo.K[0], T, a.nt[0]) - base[0],
                          tile_base(t1 + 1, a.geo.K[1], T, a.nt[1]) - base[1]};
    const int total = seg_pre[nseg];
    const int f0 = it.chunk * a.chunk;
    const int n = min(total, f0 + a.chunk) - f0;
    const int g0 = gg * kColGrids;
    const int ng = min(kColGrids, a.grids - g0);
    const int rl = lane & 15, kq = lane >> 4;
    mfma_f4 tot[ROWS][4];  // the wavefront's blocks
#pragma unroll
    for (int q = 0; q < 4 * ROWS; ++q) tot[q / 4][q % 4] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    // trajectory (or window record) and values of this lane's next sample,
    // loaded one batch ahead
    float pom[TAB ? 1 : 2];
    float4 prec[TAB ? table_f4(2, NJ) : 1];
    float2 pv[kColGrids];
    bool pvalid = false;
    int cursor = 0;
    auto fetch = [&](int b) {
        const int s_idx = b + lane;
        pvalid = s_idx < n;
        const int sg = batch_segment(seg_pre, nseg, cursor, f0 + b, 64, f0 + s_idx);
        if (pvalid) {
            const int64_t i = seg_lo[sg] + (f0 + s_idx - seg_pre[sg]);
            if constexpr (TAB) {
                load_window_record<NJ, 2>(a.geo, i, prec);
            } else {
#pragma unroll
                for (int ax = 0; ax < 2; ++ax) pom[ax] = a.om_sorted[i * 2 + ax];
            }
            const float2 *y = a.y + int64_t(g0) * a.M + (a.y_sorted ? i : int64_t(a.perm[i]));
#pragma unroll
            for (int q = 0; q < kColGrids; ++q) pv[q] = q < ng ? y[int64_t(q) * a.M] : make_float2(0.f, 0.f);
        }
    };
    fetch(wave * 64);
    for (int b0 = 0; b0 < n; b0 += NW * 64) {
        {
            float4 *z = reinterpret_cast<float4 *>(rec + wave * 64 * RS);
            for (int e = lane; e < 16 * RS; e += 64) z[e] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        group_sync(64);
        // ---- stage this lane's sample
        unsigned mk = 0;
        float2 ph = make_float2(1.f, 0.f);
        if constexpr (!TAB)
            if (pvalid && a.geo.minmax) ph = mm_phase<2>(a.geo, pom);
#pragma unroll
        for (int q = 0; q < kColGrids; ++q) {
            const float2 v = pvalid ? (a.geo.minmax ? cmulcj(ph, pv[q]) : pv[q]) : make_float2(0.f, 0.f);
            val[int(threadIdx.x) * VS + 2 * q] = v.x;
            val[int(threadIdx.x) * VS + 2 * q + 1] = v.y;
        }
        if (pvalid) {
            float *my = rec + int(threadIdx.x) * RS;
            int kwa[2];
            float wva[2][NJ];
            if constexpr (TAB)
                unpack_window<NJ, 2>(prec, kwa, wva);
            else
                eval_window<NJ, 2>(a.geo, pom, kwa, wva);
            unsigned bm[2] = {0u, 0u};
#pragma unroll
            for (int ax = 0; ax < 2; ++ax) {
                const int K = a.geo.K[ax];
                float *wv = wva[ax];
                if (a.geo.minmax) mm_sign_taps<NJ>(wv, K - kwa[ax]);
                // first tap relative to the tile; windows wrapping in from the
                // top of the axis come in negative (an axis of one tile wraps
                // inside it instead)
                int o = kwa[ax] - base[ax];
                const bool one = a.nt[ax] == 1;
                if (!one && o >= T) o -= K;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    int x = o + j;
                    if (one && x >= K) x -= K;
                    const bool in = unsigned(x) < unsigned(T) && j < J;
                    my[in ? ax * T + x : 2 * T] = wv[j];
                    bm[ax] |= in ? 1u << (x >> 2) : 0u;
                }
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if ((bm[0] >> b) & 1u) mk |= bm[1] << (4 * b);
        }
        smask[threadIdx.x] = mk;
        if (b0 + NW * 64 < n) fetch(b0 + NW * 64 + wave * 64);
        group_sync(64 * NW);
        // ---- walk: lane l looks at samples 4 l .. 4 l + 3, so 16 bits of a
        // ballot are a batch.  Two blocks side by side at a time (they share the
        // values and the row weights, and their products are independent), two
        // groups of samples per step; a batch's products are one chain, added to
        // the block's total.
        unsigned gm = 0;
        if (lane < 16 * NW) {
            const uint4 m4 = reinterpret_cast<const uint4 *>(smask)[lane];
            gm = m4.x | m4.y | m4.z | m4.w;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int row = wave * ROWS + r;
            const int a0 = 4 * row + (rl >> 2);
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const int a1 = T + 4 * q + (rl & 3);
                const uint64_t reached = __ballot(((gm >> (4 * row + q)) & 3u) != 0u);
                for (int w = 0; w < NW; ++w) {
                    uint64_t act = NW == 1 ? reached : reached & (uint64_t(0xffff) << (16 * w));
                    if (!act) continue;
                    mfma_f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
                    do {
                        const int i0 = int(__builtin_ctzll(act));
                        act &= act - 1;
                        const bool two = act != 0;
                        const int i1 = two ? int(__builtin_ctzll(act)) : i0;
                        act &= act - 1;
                        const float *s0 = rec + (4 * i0 + kq) * RS, *s1 = rec + (4 * i1 + kq) * RS;
                        const float v0 = val[(4 * i0 + kq) * VS + rl], v1 = val[(4 * i1 + kq) * VS + rl];
                        const float r0 = s0[a0], x0 = s0[a1], y0 = s0[a1 + 4], r1 = s1[a0], x1 = s1[a1], y1 = s1[a1 + 4];
                        // (left alone, the compiler waits for the first group's products
                        // before it loads the second's values: 1774 us against 1766)
                        __builtin_amdgcn_sched_barrier(0);
                        const float w1 = two ? v1 : 0.f;
                        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(r0 * x0, v0, c0, 0, 0, 0);
                        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(r0 * y0, v0, c1, 0, 0, 0);
                        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(r1 * x1, w1, c0, 0, 0, 0);
                        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(r1 * y1, w1, c1, 0, 0, 0);
                    } while (act);
                    tot[r][q] += c0;
                    tot[r][q + 1] += c1;
                }
            }
        }
        group_sync(64 * NW);
    }
    // ---- write the tile.  D[i][j] of block q sits in lane j + 16 (i / 4),
    // register i % 4: the lane holds part j & 1 of grid j / 2 at row x0 = 4
    // (q / 4) + lane / 16, columns x1 = 4 (q % 4) + register.  Neighbouring
    // lanes swap halves, so each stores two whole cells (16 bytes: tiles, grids
    // and partial tiles start at even cells).
    const bool to_partial = it.nchunks > 1;
    const int g = g0 + (rl >> 1);
    const bool odd = rl & 1;
    float2 *dst = to_partial ? a.partials + (int64_t(g) * a.n_slots + it.slot + it.chunk) * a.tile_cells
                             : a.h + int64_t(g) * a.grid_elems;
    const int64_t pitch = to_partial ? T : a.geo.K[1];
    const int64_t first = to_partial ? 0 : int64_t(base[0]) * a.geo.K[1] + base[1];
    auto swap_lane = [](float v) {  // the value of lane ^ 1
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
    };
    auto store_block = [&](int q, mfma_f4 v) {
        const float u0 = swap_lane(odd ? v[0] : v[2]), u1 = swap_lane(odd ? v[1] : v[3]);
        const float4 cells = odd ? make_float4(u0, v[2], u1, v[3]) : make_float4(v[0], u0, v[1], u1);
        const int x0 = 4 * (q >> 2) + kq, x1 = 4 * (q & 3) + (odd ? 2 : 0);
        const int64_t idx = first + x0 * pitch + x1;
        if (g - g0 < ng && (to_partial || (x0 < width[0] && x1 < width[1]))) *reinterpret_cast<float4 *>(dst + idx) = cells;
    };
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int q = 0; q < 4; ++q) store_block(4 * (wave * ROWS + r) + q, tot[r][q]);
    }
}

template <int NJ, bool TAB, int NW>
__global__ __launch_bounds__(64 * NW) void k_grid_cols(GridArgs a) {
    grid_cols_body<NJ, TAB, NW>(a, blockIdx.x, blockIdx.y);
}

template <int NJ, bool TAB, int NW>
__global__ __launch_bounds__(64 * NW) void k_grid_cols_multi(const GridArgs *__restrict__ jobs,
                                                        const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    grid_cols_body<NJ, TAB, NW>(jobs[b.x], b.y, b.z);
}

// V^H on the matrix cores in 3D, by blocks.  The tile is T0 x T1 x 16 (T0,
// T1 in {8, 16}, at most 8 blocks); its leading axes are cut into 4 x 4
// blocks, and a block with the 16 cells of the last axis is one 16 x 16
// product over the samples:
//   H[(x0, x1)][x2] = sum_s (v_s w0_s[x0] w1_s[x1]) w2_s[x2]
// (v_mfma_f32_16x16x4_f32, samples as the reduction dimension, real and
// imaginary parts sharing the w2 operand).  Each wavefront stages its own 64
// samples of a batch (value and per-axis weights spread over the tile's
// coordinates, out-of-tile taps to a discard slot, and the set of blocks the
// window reaches) and walks them four at a time over the blocks in
// registers, running only the products of blocks that one of the four
// reaches.  Wavefronts synchronise only with themselves until the end, where
// their tiles are summed in wave order (the result does not depend on
// scheduling).  With NW = 1 a work item is one wavefront, which writes its
// blocks straight from registers (no summation across wavefronts).
template <int NJ, int T0, int T1, bool TAB, int NW>
__device__ __forceinline__ void grid_blk_body(const GridArgs &a, int64_t item, int g) {
    constexpr int T2 = 16;
    constexpr int NB1 = T1 / 4;
    constexpr int NBLK = (T0 / 4) * NB1;
    constexpr int TRASH = 2;  // discard slot of a record
    constexpr int ROW[3] = {3, 3 + T0, 3 + T0 + T1};
    constexpr int TAX[3] = {T0, T1, T2};
    constexpr int RS = 3 + T0 + T1 + T2;  // floats per record (odd)
    constexpr int CELLS = T0 * T1 * T2;
    static_assert(RS % 2 == 1 && NBLK >= 4 && NBLK <= 8, "tile shape");
    extern __shared__ float blk_lds[];
    __shared__ int seg_lo[kMaxNeighbors + 1];
    __shared__ int seg_pre[kMaxNeighbors + 1];
    const GridItem it = a.items[item];
    const int nseg = grid_item_segments(a, item, seg_lo, seg_pre);
    const int J = a.geo.J;
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    float *rec = blk_lds + wave * 64 * (RS + 1);                 // [64][RS]
    unsigned *smask = reinterpret_cast<unsigned *>(rec + 64 * RS);  // [64]

    int tc[3];
    {
        int t = it.tile;
#pragma unroll
        for (int ax = 2; ax >= 0; --ax) {
            tc[ax] = t % a.nt[ax];
            t /= a.nt[ax];
        }
    }
    const int base[3] = {tile_base(tc[0], a.geo.K[0], T0, a.nt[0]), tile_base(tc[1], a.geo.K[1], T1, a.nt[1]),
                         tile_base(tc[2], a.geo.K[2], T2, a.nt[2])};
    const int total = seg_pre[nseg];
    const int f0 = it.chunk * a.chunk;
    const int n = min(total, f0 + a.chunk) - f0;

    // walk roles: lane rl + 16 kq reads row rl of sample kq's A operand and
    // column rl of its B operand; block q covers x0 in 4 (q / NB1) + [0, 4),
    // x1 in 4 (q % NB1) + [0, 4), its row rl is (x0, x1) = (+rl / 4, +rl % 4)
    const int rl = lane & 15;
    const int kq = lane >> 4;
    const float2 *y = a.y + int64_t(g) * a.M;
    mfma_f4 acc_re[NBLK], acc_im[NBLK];
#pragma unroll
    for (int q = 0; q < NBLK; ++q) {
        acc_re[q] = mfma_f4{0.f, 0.f, 0.f, 0.f};
        acc_im[q] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    }
    // trajectory (or window record) and value of this lane's next sample,
    // loaded one batch ahead
    float pom[TAB ? 1 : 3];
    float4 prec[TAB ? table_f4(3, NJ) : 1];
    float2 pv = make_float2(0.f, 0.f);
    bool pvalid = false;
    int cursor = 0;
    auto fetch = [&](int b) {
        const int s_idx = b + wave * 64 + lane;
        pvalid = s_idx < n;
        const int sg = batch_segment(seg_pre, nseg, cursor, f0 + b + wave * 64, 64, f0 + s_idx);
        if (pvalid) {
            const int64_t i = seg_lo[sg] + (f0 + s_idx - seg_pre[sg]);
            if constexpr (TAB) {
                load_window_record<NJ, 3>(a.geo, i, prec);
            } else {
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) pom[ax] = a.om_sorted[i * 3 + ax];
            }
            pv = a.y_sorted ? y[i] : y[a.perm[i]];
        }
    };
    fetch(0);
    for (int b0 = 0; b0 < n; b0 += 64 * NW) {
        {
            float4 *z = reinterpret_cast<float4 *>(rec);
            for (int e = lane; e < 16 * RS; e += 64) z[e] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        group_sync(64);
        // ---- stage this lane's sample
        unsigned mk = 0;
        if (pvalid) {
            float *my = rec + lane * RS;
            if constexpr (!TAB)
                if (a.geo.minmax) pv = cmulcj(mm_phase<3>(a.geo, pom), pv);
            my[0] = pv.x;
            my[1] = pv.y;
            unsigned bm[2] = {0u, 0u};
            int kwa[3];
            float wta[TAB ? 3 : 1][NJ];
            if constexpr (TAB) unpack_window<NJ, 3>(prec, kwa, wta);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int K = a.geo.K[ax];
                float wv[NJ];
                int kw;
                if constexpr (TAB) {
                    kw = kwa[ax];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) wv[j] = wta[ax][j];
                } else {
                    const double u = __dmul_rn(double(pom[ax]), a.geo.C[ax]);
                    const double k0 = floor(u - 0.5 * J) + 1.0;
                    const float fr = float(u - k0 - (0.5 * J - 1.0));
                    kw = wrap_first_tap(k0, K);
                    poly_rows<NJ>(a.geo.coef[ax], a.geo.jp, a.geo.nq[ax], 2.0f * fr - 1.0f, wv);
                    if (a.geo.minmax) mm_sign_taps<NJ>(wv, K - kw);
                }
                if (a.nt[ax] > 1) {
                    // first tap relative to the tile, in [-(J-1), T): a window
                    // wrapping in from the top of the axis comes in negative
                    int o = kw - base[ax];
                    if (o >= TAX[ax]) o -= K;
                    // taps past J carry zero weights (zero coefficient rows)
                    // and land outside the window: harmless either way
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const int x = o + j;
                        my[unsigned(x) < unsigned(TAX[ax]) ? ROW[ax] + x : TRASH] = wv[j];
                    }
                    if (ax < 2) {
                        // blocks of 4 cells the window's cells in the tile fall in
                        const int c0 = max(o, 0), c1 = min(o + J - 1, TAX[ax] - 1);
                        bm[ax] = c0 <= c1 ? ((2u << (c1 >> 2)) - 1u) & ~((1u << (c0 >> 2)) - 1u) : 0u;
                    }
                } else {
                    // the axis is one tile: taps wrap around inside it
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        int x = kw + j;
                        if (x >= K) x -= K;
                        const bool in = j < J;
                        my[in ? ROW[ax] + x : TRASH] = wv[j];
                        if (ax < 2) bm[ax] |= in ? 1u << (x >> 2) : 0u;
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < T0 / 4; ++b)
                if ((bm[0] >> b) & 1u) mk |= bm[1] << (b * NB1);
        }
        smask[lane] = mk;
        if (b0 + 64 * NW < n) fetch(b0 + 64 * NW);
        group_sync(64);
        // ---- walk: lane l < 16 looks at samples 4l .. 4l + 3 (one product's
        // worth) and the blocks they reach.  Block by block, the wavefront
        // runs the products with work for that block, two at a time with all
        // their operand reads issued first (one accumulator per loop, so it
        // stays in its registers).
        unsigned gm = 0;
        if (lane < 16) {
            const uint4 m4 = reinterpret_cast<const uint4 *>(smask)[lane];
            gm = m4.x | m4.y | m4.z | m4.w;
        }
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
            const int a0 = ROW[0] + 4 * (q / NB1) + (rl >> 2);
            const int a1 = ROW[1] + 4 * (q % NB1) + (rl & 3);
            uint64_t act = __ballot((gm >> q) & 1u);
            while (act) {
                const int g0 = int(__builtin_ctzll(act));
                act &= act - 1;
                const bool two = act != 0;
                const int g1 = two ? int(__builtin_ctzll(act)) : g0;
                act &= act - 1;
                const float *s0 = rec + (4 * g0 + kq) * RS;
                const float *s1 = rec + (4 * g1 + kq) * RS;
                const float vx0 = s0[0], vy0 = s0[1], b0w = s0[ROW[2] + rl], l0 = s0[a0] * s0[a1];
                const float vx1 = s1[0], vy1 = s1[1], b1w = s1[ROW[2] + rl], l1 = two ? s1[a0] * s1[a1] : 0.f;
                acc_re[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx0 * l0, b0w, acc_re[q], 0, 0, 0);
                acc_im[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(vy0 * l0, b0w, acc_im[q], 0, 0, 0);
                acc_re[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx1 * l1, b1w, acc_re[q], 0, 0, 0);
                acc_im[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(vy1 * l1, b1w, acc_im[q], 0, 0, 0);
            }
        }
        group_sync(64);
    }
    // ---- write the tile.  D[i][j] of block q sits in lane j + 16 (i / 4),
    // register i % 4, block row i being (x0, x1) = (4 (q / NB1) + i / 4,
    // 4 (q % NB1) + i % 4).
    const bool to_partial = it.nchunks > 1;
    float2 *dst = to_partial ? a.partials + (int64_t(g) * a.n_slots + it.slot + it.chunk) * a.tile_cells
                             : a.h + int64_t(g) * a.grid_elems;
    const int64_t K1 = a.geo.K[1], K2 = a.geo.K[2];
    // the tile's own cells (partial tiles are stored whole)
    const int w0 = to_partial ? T0 : tile_base(tc[0] + 1, a.geo.K[0], T0, a.nt[0]) - base[0];
    const int w1 = to_partial ? T1 : tile_base(tc[1] + 1, a.geo.K[1], T1, a.nt[1]) - base[1];
    const int w2 = to_partial ? T2 : tile_base(tc[2] + 1, a.geo.K[2], T2, a.nt[2]) - base[2];
    if constexpr (NW == 1) {
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
            const int x0 = 4 * (q / NB1) + kq;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int x1 = 4 * (q % NB1) + r;
                const int64_t idx = to_partial ? int64_t((x0 * T1 + x1) * T2 + rl)
                                               : (int64_t(base[0] + x0) * K1 + base[1] + x1) * K2 + base[2] + rl;
                if (x0 < w0 && x1 < w1 && rl < w2) dst[idx] = make_float2(acc_re[q][r], acc_im[q][r]);
            }
        }
        return;
    }
    // several wavefronts: their tiles are summed in wave order
    __syncthreads();  // every wave is done with its staging area
    float2 *red = reinterpret_cast<float2 *>(blk_lds);  // [4][CELLS], reuses the staging LDS
#pragma unroll
    for (int q = 0; q < NBLK; ++q) {
        const int x0 = 4 * (q / NB1) + kq;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x1 = 4 * (q % NB1) + r;
            red[wave * CELLS + (x0 * T1 + x1) * T2 + rl] = make_float2(acc_re[q][r], acc_im[q][r]);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < CELLS; e += 64 * NW) {
        float2 sum = red[e];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum = cadd(sum, red[w * CELLS + e]);
        const int x2 = e % T2, x1 = (e / T2) % T1, x0 = e / (T1 * T2);
        const int64_t idx = to_partial ? int64_t(e) : (int64_t(base[0] + x0) * K1 + base[1] + x1) * K2 + base[2] + x2;
        if (x0 < w0 && x1 < w1 && x2 < w2) dst[idx] = sum;
    }
}

template <int NJ, int T0, int T1, bool TAB, int NW>
__global__ __launch_bounds__(64 * NW) void k_grid_blk(GridArgs a) {
    grid_blk_body<NJ, T0, T1, TAB, NW>(a, blockIdx.x, blockIdx.y);
}

template <int NJ, int T0, int T1, bool TAB, int NW>
__global__ __launch_bounds__(64 * NW) void k_grid_blk_multi(const GridArgs *__restrict__ jobs,
                                                           const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    grid_blk_body<NJ, T0, T1, TAB, NW>(jobs[b.x], b.y, b.z);
}

// Sums the partial tiles of every split tile; one workgroup per (tile,
// kReduceCellsPerWg cells, grid).  The kReduceLanes threads of a cell each
// sum every kReduceLanes-th partial tile in chunk order, and their sums are
// added in lane order (the order of the first inverse FFT pass that sums
// them itself), so the dependent chain of loads of the most crowded tiles is
// kReduceLanes times shorter.
__device__ __forceinline__ void reduce_partials_body(const ReduceArgs &a, int64_t hot, int cb, int g) {
    __shared__ float2 lane_sum[kReduceLanes][kReduceCellsPerWg];
    const HotTile ht = a.hot[hot];
    const int cl = int(threadIdx.x) % kReduceCellsPerWg;  // cell of the block
    const int ln = int(threadIdx.x) / kReduceCellsPerWg;  // its lane
    const int e = cb * kReduceCellsPerWg + cl;
    float2 acc = make_float2(0.f, 0.f);
    if (e < a.tile_cells) {
        const float2 *p = a.partials + (int64_t(g) * a.n_slots + ht.slot) * a.tile_cells + e;
        constexpr int R = 8;  // partial tiles in flight per round trip
        for (int c0 = ln; c0 < ht.nchunks; c0 += R * kReduceLanes) {
            float2 t[R];
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (c0 + j * kReduceLanes < ht.nchunks) t[j] = p[int64_t(c0 + j * kReduceLanes) * a.tile_cells];
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (c0 + j * kReduceLanes < ht.nchunks) acc = cadd(acc, t[j]);
        }
    }
    lane_sum[ln][cl] = acc;
    __syncthreads();
    if (ln != 0 || e >= a.tile_cells) return;
#pragma unroll
    for (int j = 1; j < kReduceLanes; ++j) acc = cadd(acc, lane_sum[j][cl]);
    int tc[kMaxDim];
    {
        int t = ht.tile;
        for (int ax = a.d - 1; ax >= 0; --ax) {
            tc[ax] = t % a.nt[ax];
            t /= a.nt[ax];
        }
    }
    int rem = e;
    int l[kMaxDim];
    for (int ax = a.d - 1; ax >= 0; --ax) {
        l[ax] = rem % a.T[ax];
        rem /= a.T[ax];
    }
    int64_t idx = 0;
    for (int ax = 0; ax < a.d; ++ax) {
        const int k = tile_base(tc[ax], a.K[ax], a.T[ax], a.nt[ax]) + l[ax];
        if (k >= tile_base(tc[ax] + 1, a.K[ax], a.T[ax], a.nt[ax])) return;  // past the tile's own cells
        idx = idx * a.K[ax] + k;
    }
    a.h[int64_t(g) * a.grid_elems + idx] = acc;
}

__global__ __launch_bounds__(256) void k_reduce_partials(ReduceArgs a) {
    reduce_partials_body(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

__global__ __launch_bounds__(256) void k_reduce_partials_multi(const ReduceArgs *__restrict__ jobs,
                                                             const int4 *__restrict__ blocks) {
    const int4 b = blocks[blockIdx.x];
    reduce_partials_body(jobs[b.x], b.y, b.z, b.w);
}

}  // namespace

// ------------------------------------------------------------ launchers
template <int DIM, int LS>
hipError_t launch_grid_t(const GridArgs &a, hipStream_t s) {
    const size_t lds = grid_lds(a);
    const dim3 grid(unsigned(a.n_items), unsigned(a.grids));
    if (a.geo.jp == 8)
        launch_kernel((k_grid<DIM, LS, 8>), grid, dim3(kGridThreads), lds, s, a);
    else if (a.geo.jp == 16)
        launch_kernel((k_grid<DIM, LS, 16>), grid, dim3(kGridThreads), lds, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int DIM>
hipError_t launch_grid_d(const GridArgs &a, hipStream_t s) {
    switch (a.seg_len) {
        case 4: return launch_grid_t<DIM, 4>(a, s);
        case 8: return launch_grid_t<DIM, 8>(a, s);
        case 16: return launch_grid_t<DIM, 16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// The window-table form of the sample kernels exists for windows of up to 8
// taps (table_taps 6 or 8); wider windows evaluate the kernel on the fly even
// when the plan holds a table.
inline bool use_table(const SampleGeom &g) { return g.wtab != nullptr && table_taps(g.J) <= 8; }

template <int DIM, int NJ, int MB, bool TAB>
hipError_t launch_grid_mfma_t(const GridArgs &a, hipStream_t s) {
    const size_t lds = grid_lds(a);
    const int gp = a.grids_per_wg;
    const dim3 grid(unsigned(a.n_items), unsigned((a.grids + gp - 1) / gp));
    switch (gp) {
        case 1: launch_kernel((k_grid_mfma<DIM, NJ, MB, 1, TAB>), grid, dim3(256), lds, s, a); break;
        case 2: launch_kernel((k_grid_mfma<DIM, NJ, MB, 2, TAB>), grid, dim3(256), lds, s, a); break;
        case 4:
            if constexpr (MB <= 2) {
                launch_kernel((k_grid_mfma<DIM, NJ, MB, 4, TAB>), grid, dim3(256), lds, s, a);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int DIM, int NJ, int MB>
hipError_t launch_grid_mfma_m(const GridArgs &a, hipStream_t s) {
    if constexpr (NJ <= 8)
        if (use_table(a.geo)) return launch_grid_mfma_t<DIM, NJ, MB, true>(a, s);
    return launch_grid_mfma_t<DIM, NJ, MB, false>(a, s);
}

template <int DIM, int NJ>
hipError_t launch_grid_mfma_j(const GridArgs &a, hipStream_t s) {
    switch (a.tile_cells) {
        case 256: return launch_grid_mfma_m<DIM, NJ, 1>(a, s);
        case 512: return launch_grid_mfma_m<DIM, NJ, 2>(a, s);
        case 1024: return launch_grid_mfma_m<DIM, NJ, 4>(a, s);
        default: return hipErrorInvalidValue;
    }
}

template <int DIM>
hipError_t launch_grid_mfma_d(const GridArgs &a, hipStream_t s) {
    if (a.T[DIM - 1] != 16) return hipErrorInvalidValue;
    // taps evaluated per sample: J rounded up to 6, 8 or 16
    if (a.geo.J <= 6) return launch_grid_mfma_j<DIM, 6>(a, s);
    if (a.geo.J <= 8) return launch_grid_mfma_j<DIM, 8>(a, s);
    return launch_grid_mfma_j<DIM, 16>(a, s);
}

template <int NJ, int T0, int T1, bool TAB, int NW, bool MULTI>
void launch_grid_blk_i(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks, size_t lds,
                       hipStream_t s) {
    if (MULTI)
        launch_kernel((k_grid_blk_multi<NJ, T0, T1, TAB, NW>), dim3(unsigned(nblocks)), dim3(64 * NW), lds, s, jobs,
                      blocks);
    else
        launch_kernel((k_grid_blk<NJ, T0, T1, TAB, NW>), dim3(unsigned(a.n_items), unsigned(a.grids)), dim3(64 * NW),
                      lds, s, a);
}

template <int NJ, int T0, int T1, bool MULTI>
hipError_t launch_grid_blk_t(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks,
                             size_t lds, hipStream_t s) {
    const bool tab = NJ <= 8 && use_table(a.geo);
    if (a.grid_waves == 1) {
        if (tab)
            launch_grid_blk_i<NJ, T0, T1, true, 1, MULTI>(a, jobs, blocks, nblocks, lds, s);
        else
            launch_grid_blk_i<NJ, T0, T1, false, 1, MULTI>(a, jobs, blocks, nblocks, lds, s);
    } else {
        if (tab)
            launch_grid_blk_i<NJ, T0, T1, true, 4, MULTI>(a, jobs, blocks, nblocks, lds, s);
        else
            launch_grid_blk_i<NJ, T0, T1, false, 4, MULTI>(a, jobs, blocks, nblocks, lds, s);
    }
    return hipGetLastError();
}

template <int NJ, bool MULTI>
hipError_t launch_grid_blk_j(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks,
                             size_t lds, hipStream_t s) {
    if (a.T[0] == 8 && a.T[1] == 8) return launch_grid_blk_t<NJ, 8, 8, MULTI>(a, jobs, blocks, nblocks, lds, s);
    if (a.T[0] == 8 && a.T[1] == 16) return launch_grid_blk_t<NJ, 8, 16, MULTI>(a, jobs, blocks, nblocks, lds, s);
    if (a.T[0] == 16 && a.T[1] == 8) return launch_grid_blk_t<NJ, 16, 8, MULTI>(a, jobs, blocks, nblocks, lds, s);
    return hipErrorInvalidValue;
}

template <bool MULTI>
hipError_t launch_grid_blk(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks,
                           size_t lds, hipStream_t s) {
    if (a.geo.d != 3 || a.T[2] != 16) return hipErrorInvalidValue;
    if (a.geo.J <= 6) return launch_grid_blk_j<6, MULTI>(a, jobs, blocks, nblocks, lds, s);
    if (a.geo.J <= 8) return launch_grid_blk_j<8, MULTI>(a, jobs, blocks, nblocks, lds, s);
    return launch_grid_blk_j<16, MULTI>(a, jobs, blocks, nblocks, lds, s);
}

template <int NJ, bool TAB, int NW>
void launch_grid_cols_w(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks, size_t lds,
                        hipStream_t s) {
    const dim3 block(64 * NW);
    if (jobs)
        launch_kernel((k_grid_cols_multi<NJ, TAB, NW>), dim3(unsigned(nblocks)), block, lds, s, jobs, blocks);
    else
        launch_kernel((k_grid_cols<NJ, TAB, NW>), dim3(unsigned(a.n_items), unsigned(grid_groups(a))), block, lds, s, a);
}

template <int NJ, bool TAB>
void launch_grid_cols_t(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks, size_t lds,
                        hipStream_t s) {
    if (a.cols == 4)
        launch_grid_cols_w<NJ, TAB, 4>(a, jobs, blocks, nblocks, lds, s);
    else
        launch_grid_cols_w<NJ, TAB, 1>(a, jobs, blocks, nblocks, lds, s);
}

// One problem's launch, or (jobs != nullptr) a multi-problem one like a.
hipError_t launch_grid_cols(const GridArgs &a, const GridArgs *jobs, const int4 *blocks, int64_t nblocks, size_t lds,
                            hipStream_t s) {
    if (a.geo.d != 2 || a.T[0] != 16 || a.T[1] != 16) return hipErrorInvalidValue;
    const bool tab = use_table(a.geo);
    if (a.geo.J <= 6 && tab)
        launch_grid_cols_t<6, true>(a, jobs, blocks, nblocks, lds, s);
    else if (a.geo.J <= 6)
        launch_grid_cols_t<6, false>(a, jobs, blocks, nblocks, lds, s);
    else if (a.geo.J <= 8 && tab)
        launch_grid_cols_t<8, true>(a, jobs, blocks, nblocks, lds, s);
    else if (a.geo.J <= 8)
        launch_grid_cols_t<8, false>(a, jobs, blocks, nblocks, lds, s);
    else
        launch_grid_cols_t<16, false>(a, jobs, blocks, nblocks, lds, s);
    return hipGetLastError();
}

hipError_t launch_grid(const GridArgs &a, hipStream_t s) {
    if (a.n_items == 0) return hipSuccess;
    if (a.cols) return launch_grid_cols(a, nullptr, nullptr, 0, grid_lds(a), s);
    if (a.blk) return launch_grid_blk<false>(a, nullptr, nullptr, 0, grid_lds(a), s);
    if (a.mfma) {
        switch (a.geo.d) {
            case 2: return launch_grid_mfma_d<2>(a, s);
            case 3: return launch_grid_mfma_d<3>(a, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (a.geo.d) {
        case 1: return launch_grid_d<1>(a, s);
        case 2: return launch_grid_d<2>(a, s);
        case 3: return launch_grid_d<3>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// Kernel instance of a gridding launch: matrix cores (d, taps rounded to
// 6/8/16, row blocks) or vector ALUs (d, segment length, coefficient row
// width), as launch_grid picks it; -1 if there is none.
int grid_variant(const GridArgs &a) {
    if (a.cols) {
        if (a.geo.d != 2 || a.T[0] != 16 || a.T[1] != 16) return -1;
        return 5000 + 100 * a.cols + 10 * (a.geo.J <= 6 ? 0 : a.geo.J <= 8 ? 1 : 2) + (use_table(a.geo) ? 1 : 0);
    }
    if (a.blk) {
        if (a.geo.d != 3 || a.T[2] != 16 || (a.T[0] != 8 && a.T[0] != 16) || (a.T[1] != 8 && a.T[1] != 16) ||
            a.T[0] * a.T[1] > 128)
            return -1;
        const int nj = a.geo.J <= 6 ? 0 : a.geo.J <= 8 ? 1 : 2;
        if (a.grid_waves != 1 && a.grid_waves != 4) return -1;
        return 3000 + 100 * a.grid_waves + 10 * nj + (a.T[0] == 16 ? 2 : 0) + (a.T[1] == 16 ? 1 : 0);
    }
    if (a.mfma) {
        if (a.geo.d < 2 || a.T[a.geo.d - 1] != 16) return -1;
        const int nj = a.geo.J <= 6 ? 6 : a.geo.J <= 8 ? 8 : 16;
        const int mb = a.tile_cells / 256;
        if (a.tile_cells % 256 || (mb != 1 && mb != 2 && mb != 4)) return -1;
        const int gp = a.grids_per_wg;
        if ((gp != 1 && gp != 2 && gp != 4) || gp * mb > 8) return -1;
        return 10000 * gp + 1000 + 100 * a.geo.d + 10 * (nj == 6 ? 0 : nj == 8 ? 1 : 2) + mb;
    }
    if (a.seg_len != 4 && a.seg_len != 8 && a.seg_len != 16) return -1;
    if (a.geo.jp != 8 && a.geo.jp != 16) return -1;
    return 2000 + 100 * a.geo.d + a.seg_len * 2 + (a.geo.jp == 16 ? 1 : 0);
}

int grid_groups(const GridArgs &a) {
    const int gp = a.cols ? kColGrids : a.mfma ? a.grids_per_wg : 1;
    return (a.grids + gp - 1) / gp;
}

size_t grid_lds(const GridArgs &a) {
    if (a.cols) return size_t(64) * a.cols * ((2 * 16 + 1) + (2 * kColGrids + 1) + 1) * sizeof(float);
    if (a.blk) {
        const size_t staged = size_t(64) * a.grid_waves * (3 + a.T[0] + a.T[1] + a.T[2] + 1) * sizeof(float);
        return a.grid_waves == 1 ? staged : std::max(staged, size_t(a.grid_waves) * a.tile_cells * sizeof(float2));
    }
    if (a.mfma) {
        int tsum = 0;
        for (int ax = 0; ax < a.geo.d; ++ax) tsum += a.T[ax];
        const size_t rs = size_t((2 * a.grids_per_wg + tsum) | 1);
        return std::max(size_t(4) * 64 * rs, size_t(4) * 2 * a.tile_cells) * sizeof(float);
    }
    return size_t(kGridThreads / a.group_lanes) * a.stage_floats * sizeof(float);
}

namespace {
template <int DIM, int NJ, int MB, bool TAB>
hipError_t grid_mfma_multi_t(const GridArgs *jobs, const int4 *blocks, int64_t n, int gp, size_t lds, hipStream_t s) {
    const dim3 grid = dim3(unsigned(n));
    switch (gp) {
        case 1: launch_kernel((k_grid_mfma_multi<DIM, NJ, MB, 1, TAB>), grid, dim3(256), lds, s, jobs, blocks); break;
        case 2: launch_kernel((k_grid_mfma_multi<DIM, NJ, MB, 2, TAB>), grid, dim3(256), lds, s, jobs, blocks); break;
        case 4:
            if constexpr (MB <= 2) {
                launch_kernel((k_grid_mfma_multi<DIM, NJ, MB, 4, TAB>), grid, dim3(256), lds, s, jobs, blocks);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int DIM, int NJ, int MB>
hipError_t grid_mfma_multi_m(const GridArgs *jobs, const int4 *blocks, int64_t n, int gp, bool tab, size_t lds,
                             hipStream_t s) {
    if constexpr (NJ <= 8)
        if (tab) return grid_mfma_multi_t<DIM, NJ, MB, true>(jobs, blocks, n, gp, lds, s);
    return grid_mfma_multi_t<DIM, NJ, MB, false>(jobs, blocks, n, gp, lds, s);
}

template <int DIM, int NJ>
hipError_t grid_mfma_multi_j(const GridArgs *jobs, const int4 *blocks, int64_t n, int mb, int gp, bool tab,
                             size_t lds, hipStream_t s) {
    switch (mb) {
        case 1: return grid_mfma_multi_m<DIM, NJ, 1>(jobs, blocks, n, gp, tab, lds, s);
        case 2: return grid_mfma_multi_m<DIM, NJ, 2>(jobs, blocks, n, gp, tab, lds, s);
        case 4: return grid_mfma_multi_m<DIM, NJ, 4>(jobs, blocks, n, gp, tab, lds, s);
        default: return hipErrorInvalidValue;
    }
}

template <int DIM>
hipError_t grid_mfma_multi_d(const GridArgs *jobs, const int4 *blocks, int64_t n, const GridArgs &p, size_t lds,
                             hipStream_t s) {
    const int mb = p.tile_cells / 256;
    const bool tab = use_table(p.geo);
    if (p.geo.J <= 6) return grid_mfma_multi_j<DIM, 6>(jobs, blocks, n, mb, p.grids_per_wg, tab, lds, s);
    if (p.geo.J <= 8) return grid_mfma_multi_j<DIM, 8>(jobs, blocks, n, mb, p.grids_per_wg, tab, lds, s);
    return grid_mfma_multi_j<DIM, 16>(jobs, blocks, n, mb, p.grids_per_wg, tab, lds, s);
}

template <int DIM, int LS>
hipError_t grid_valu_multi_t(const GridArgs *jobs, const int4 *blocks, int64_t n, int jp, size_t lds, hipStream_t s) {
    if (jp == 8)
        launch_kernel((k_grid_multi<DIM, LS, 8>), dim3(unsigned(n)), dim3(kGridThreads), lds, s, jobs, blocks);
    else if (jp == 16)
        launch_kernel((k_grid_multi<DIM, LS, 16>), dim3(unsigned(n)), dim3(kGridThreads), lds, s, jobs, blocks);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int DIM>
hipError_t grid_valu_multi_d(const GridArgs *jobs, const int4 *blocks, int64_t n, const GridArgs &p, size_t lds,
                             hipStream_t s) {
    switch (p.seg_len) {
        case 4: return grid_valu_multi_t<DIM, 4>(jobs, blocks, n, p.geo.jp, lds, s);
        case 8: return grid_valu_multi_t<DIM, 8>(jobs, blocks, n, p.geo.jp, lds, s);
        case 16: return grid_valu_multi_t<DIM, 16>(jobs, blocks, n, p.geo.jp, lds, s);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t launch_grid_multi(const GridArgs *jobs, const int4 *blocks, int64_t nblocks, const GridArgs &proto,
                             size_t lds, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    if (grid_variant(proto) < 0) return hipErrorInvalidValue;
    if (proto.cols) return launch_grid_cols(proto, jobs, blocks, nblocks, lds, s);
    if (proto.blk) return launch_grid_blk<true>(proto, jobs, blocks, nblocks, lds, s);
    if (proto.mfma) {
        switch (proto.geo.d) {
            case 2: return grid_mfma_multi_d<2>(jobs, blocks, nblocks, proto, lds, s);
            case 3: return grid_mfma_multi_d<3>(jobs, blocks, nblocks, proto, lds, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (proto.geo.d) {
        case 1: return grid_valu_multi_d<1>(jobs, blocks, nblocks, proto, lds, s);
        case 2: return grid_valu_multi_d<2>(jobs, blocks, nblocks, proto, lds, s);
        case 3: return grid_valu_multi_d<3>(jobs, blocks, nblocks, proto, lds, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_reduce_partials_multi(const ReduceArgs *jobs, const int4 *blocks, int64_t nblocks, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    launch_kernel(k_reduce_partials_multi, dim3(unsigned(nblocks)), dim3(256), 0, s, jobs, blocks);
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const ReduceArgs &a, hipStream_t s) {
    if (a.n_hot == 0) return hipSuccess;
    launch_kernel(k_reduce_partials,
                  dim3(unsigned(a.n_hot), unsigned((a.tile_cells + kReduceCellsPerWg - 1) / kReduceCellsPerWg),
                       unsigned(a.grids)),
                  dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace nufft
