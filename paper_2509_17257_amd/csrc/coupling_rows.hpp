// Coupling stage of the FP64 operator for any rank k > 32 on the matrix cores:
//   y_t = sum_{(t,s) in C_t, admissible} S_b x_s     for every row cluster t.
//
// A work-group owns 64 rows of y_t (four waves of 16) and a slab of 16 NJ columns; the
// contraction over a block runs in chunks of 64 columns of S_b, whose 64 rows of x_s go
// through LDS (double-buffered) while each wave streams its 16 x 64 slice of S_b into
// registers in operand order (s_index layout 1, rows padded to 16 and columns to 8 with
// zeros).  Everything is loaded one chunk ahead from clamped addresses.  The row groups and
// column slabs of a row cluster are consecutive work-groups of one XCD, so that they share x_s
// and S_b in its L2.
//
// Bound by the stream of S (8 k^2 bytes against 2 k^2 m flops per block): rank 125, 16 columns,
// 32768 points on a sphere, leaf 128: 0.377 ms, 5.9 TB/s of S; the LDS-tiled vector kernel that
// served these ranks before took 3.106 ms, 0.7 TB/s.
#pragma once

#include <algorithm>
#include <type_traits>

#include "device.hpp"

namespace h2x {

typedef double dbl4 __attribute__((ext_vector_type(4)));

template <int NJ>
__global__ __launch_bounds__(256) void k_coupling_rows(int k, int64_t m, int32_t C, int32_t rows_per_xcd,
                                                       const int32_t *__restrict__ order,
                                                       const int64_t *__restrict__ adm_ptr,
                                                       const int32_t *__restrict__ adm_col,
                                                       const double *__restrict__ S, int64_t s_blk,
                                                       const double *__restrict__ xh, double *__restrict__ yh,
                                                       int64_t ldh, Skip skip) {
    constexpr int MC = 16 * NJ, LDX = MC + 1, XPT = 4 * NJ;
    typedef double dbl2 __attribute__((ext_vector_type(2)));
    __shared__ double xs[2][64 * LDX];
    const int nslab = (int)((m + MC - 1) / MC), ngrp = (k + 63) >> 6;
    const int qx = blockIdx.x >> 3, part = qx % (nslab * ngrp);
    const int slot = (blockIdx.x & 7) * rows_per_xcd + qx / (nslab * ngrp);
    if (slot >= C) return;
    const int32_t t = order[slot];
    if (skip(t)) return;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t j0 = (int64_t)(part % nslab) * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    const int64_t b0 = adm_ptr[t], b1 = adm_ptr[t + 1];
    const int tile = 4 * (part / nslab) + w, ktile = (k + 15) >> 4;  // 16-row tile of this wave
    const int kpair = (k + 7) >> 3, nch = (k + 63) >> 6;             // 8-column pairs, 64-column chunks

    dbl4 acc[NJ];
#pragma unroll
    for (int J = 0; J < NJ; ++J) acc[J] = dbl4{0.0, 0.0, 0.0, 0.0};

    if (b1 > b0) {
        double xv[XPT];
        dbl2 sa[8], sn[8];
        auto load = [&](int64_t b, int c, dbl2 (&dst)[8]) {
            const double *src = xh + (int64_t)adm_col[b] * k * ldh + j0;
#pragma unroll
            for (int u = 0; u < XPT; ++u) {
                const int e = tid + 256 * u, r = e / MC, col = e % MC;
                xv[u] = src[(int64_t)min(64 * c + r, k - 1) * ldh + (col < mc ? col : 0)];
            }
            // pairs past the last read the next tile's (never multiplied) or, past the block, zeros
            const __amdgpu_buffer_rsrc_t rs = buf_rsrc(S + b * s_blk, (uint32_t)(s_blk * 8));
            const uint32_t base = 16u * ((uint32_t)(min(tile, ktile - 1) * kpair + 8 * c) * 64 + lane);
#pragma unroll
            for (int q = 0; q < 8; ++q) dst[q] = __builtin_bit_cast(dbl2, buf_ld16<kBufNT>(rs, base + 1024u * q));
        };
        auto store = [&](int buf, int c) {
#pragma unroll
            for (int u = 0; u < XPT; ++u) {
                const int e = tid + 256 * u, r = e / MC, col = e % MC;
                xs[buf][r * LDX + col] = (64 * c + r < k && col < mc) ? xv[u] : 0.0;
            }
        };
        auto multiply = [&](int buf, int c) {
            const double *xb = xs[buf] + lq * LDX + lr;
            const int np = min(8, kpair - 8 * c);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < np) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int J = 0; J < NJ; ++J)
                            acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? sa[q].y : sa[q].x,
                                                                          xb[(8 * q + 4 * h) * LDX + 16 * J], acc[J], 0,
                                                                          0, 0);
                }
            }
        };
        // the list in four consecutive parts whose sums are added in order, as in every coupling
        // form of this operator (the tile form gives a part to each wave): the same bits from each
        const int quarter = (int)((b1 - b0 + 3) / 4);
        dbl4 sum[NJ];
#pragma unroll
        for (int J = 0; J < NJ; ++J) sum[J] = dbl4{0.0, 0.0, 0.0, 0.0};
        int c = 0, buf = 0, left = quarter;
        int64_t b = b0;
        load(b, 0, sa);
        store(0, 0);
        __syncthreads();
        for (;;) {
            const int cn = c + 1 < nch ? c + 1 : 0;
            const int64_t bn = cn ? b : b + 1;
            if (bn >= b1) break;
            load(bn, cn, sn);
            multiply(buf, c);
            if (__builtin_expect(!cn && --left == 0, 0)) {
                left = quarter;
#pragma unroll
                for (int J = 0; J < NJ; ++J) {
                    sum[J] += acc[J];
                    acc[J] = dbl4{0.0, 0.0, 0.0, 0.0};
                }
            }
            store(buf ^ 1, cn);
#pragma unroll
            for (int q = 0; q < 8; ++q) sa[q] = sn[q];
            __syncthreads();
            b = bn;
            c = cn;
            buf ^= 1;
        }
        multiply(buf, c);
#pragma unroll
        for (int J = 0; J < NJ; ++J) acc[J] = sum[J] + acc[J];
    }
    if (tile >= ktile) return;
    // D layout of the 16x16x4 f64 MFMA: lane l, register r -> row l / 16 + 4 r, column l % 16
#pragma unroll
    for (int J = 0; J < NJ; ++J) {
        const int col = 16 * J + lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * tile + lq + 4 * r;
            if (col < mc && row < k) yh[((int64_t)t * k + row) * ldh + j0 + col] = acc[J][r];
        }
    }
}

// The same stage for few row clusters, where one work-group per row leaves most of the chip idle
// and a list is a serial chain of load latencies: a work-group takes one 16-row tile of y_t and a
// slab of 16 columns, each of its four waves a quarter of the list, and the sums of the quarters are
// added in order.  Both operands go straight into matrix-core registers (S_b in operand order,
// x_s 16 columns by 4 rows an instruction), three 32-column steps ahead (36 loads: the wait
// counter holds 63), with no LDS and no barrier in the loop.  x_s is read once per tile instead
// of once per 64 rows, which costs more than the spreading gains once the tiles fill the chip
// (figures at coupling_in_tiles).
static __global__ __launch_bounds__(256) void k_coupling_tile(int k, int64_t m, int32_t C, int32_t rows_per_xcd,
                                                              const int32_t *__restrict__ order,
                                                              const int64_t *__restrict__ adm_ptr,
                                                              const int32_t *__restrict__ adm_col,
                                                              const double *__restrict__ S, int64_t s_blk,
                                                              const double *__restrict__ xh, double *__restrict__ yh,
                                                              int64_t ldh, Skip skip, int jpass) {
    typedef double dbl2 __attribute__((ext_vector_type(2)));
    __shared__ double red[3 * 256];
    const int nslab = (int)((m + 15) / 16), ktile = (k + 15) >> 4;
    const int unit = (int)(blockIdx.x >> 3), part = unit % (nslab * ktile);
    const int slot = (blockIdx.x & 7) * rows_per_xcd + unit / (nslab * ktile);
    if (slot >= C) return;
    const int32_t t = order[slot];
    if (skip(t)) return;
    const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = part / nslab;
    const int64_t j0 = (int64_t)(part % nslab) * 16;
    const int mc = (int)min<int64_t>(16, m - j0);
    const int nb = (int)(adm_ptr[t + 1] - adm_ptr[t]), quarter = (nb + 3) / 4;
    const int64_t b0 = adm_ptr[t] + min(nb, w * quarter), b1 = adm_ptr[t] + min(nb, (w + 1) * quarter);
    const int kpair = (k + 7) >> 3, nch = (kpair + 3) >> 2;

    dbl4 acc = dbl4{0.0, 0.0, 0.0, 0.0};
    struct Set {
        dbl2 s[4];
        double x[8];
        int lim;
    };
    // jpass: column c takes its partner c ^ 1 (J x = (-im, re) per complex column)
    const int cx = (lr < mc ? lr : 0) ^ jpass;
    const bool neg = jpass & ~lr & 1;
    if (b1 > b0) {
        // the next step to load: chunk c of block b, whose column cluster is s (past the list it
        // re-reads the last block and multiplies zeros)
        const int64_t steps = (b1 - b0) * nch;
        int64_t b = b0, left = steps;
        int c = 0;
        int32_t s = adm_col[b0], s_next = adm_col[min(b0 + 1, b1 - 1)];
        auto load = [&](Set &R) {
            // pairs past the last read the next tile's (never multiplied) or, past the block, zeros
            const __amdgpu_buffer_rsrc_t rs = buf_rsrc(S + b * s_blk, (uint32_t)(s_blk * 8));
            const uint32_t base = 16u * ((uint32_t)(tile * kpair + 4 * c) * 64 + lane);
#pragma unroll
            for (int q = 0; q < 4; ++q) R.s[q] = __builtin_bit_cast(dbl2, buf_ld16<kBufNT>(rs, base + 1024u * q));
            const double *src = xh + (int64_t)s * k * ldh + j0 + cx;
#pragma unroll
            for (int u = 0; u < 8; ++u) R.x[u] = src[(int64_t)min(32 * c + 4 * u + lq, k - 1) * ldh];
            R.lim = left > 0 ? k - 32 * c : 0;  // columns of S_b from this chunk on; none past the list
            --left;
            const bool wrap = c + 1 == nch;
            c = wrap ? 0 : c + 1;
            if (wrap) {
                b = min(b + 1, b1 - 1);
                s = s_next;
                s_next = adm_col[min(b + 1, b1 - 1)];
            }
        };
        auto multiply = [&](const Set &R) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    // zero rows of x past k (a partial last chunk: pairs past the last, too)
                    const double v = neg ? -R.x[2 * q + h] : R.x[2 * q + h];
                    const bool in = 8 * q + 4 * h + lq < R.lim;
                    const double a = h ? R.s[q].y : R.s[q].x;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? a : 0.0, in ? v : 0.0, acc, 0, 0, 0);
                }
        };
        Set r0, r1, r2, r3;  // four register sets in turn; one exit, so that the wait counts hold
        load(r0);
        load(r1);
        load(r2);
        for (int64_t i = 0; i < steps; i += 4) {
            load(r3);
            multiply(r0);
            load(r0);
            multiply(r1);
            load(r1);
            multiply(r2);
            load(r2);
            multiply(r3);
        }
    }
    if (w > 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((w - 1) * 4 + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (w > 0) return;
#pragma unroll
    for (int g = 0; g < 3; ++g)  // (an empty quarter adds zeros)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += red[(g * 4 + r) * 64 + lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * tile + lq + 4 * r;
        if (lr < mc && row < k) {
            double *y = &yh[((int64_t)t * k + row) * ldh + j0 + lr];
            *y = jpass ? *y + acc[r] : acc[r];
        }
    }
}

// whether the tile form runs: up to about six 16-row tiles per CU (rank 64, 16 columns: 193 rows
// 62 -> 42 us, cube of 359 rows 82 -> 66, sphere of 375 rows 70 -> 75; rank 125: 97 rows 85 -> 48,
// 189 rows 136 -> 93, 381 rows 198 -> 227)
inline bool coupling_in_tiles(int k, int64_t m, int32_t nrows) {
    return (int64_t)nrows * ((k + 15) / 16) * ((m + 15) / 16) <= (k > 64 ? 1600 : 1480);
}

// nrows clusters in the order of rows
inline void launch_coupling_tile(const DevMat &dm, int64_t m, const double *S, const double *xh, double *yh,
                                 int64_t ldh, hipStream_t st, Skip skip, int32_t nrows, const int32_t *rows,
                                 int jpass) {
    if (nrows <= 0) return;
    const int32_t rpx = (nrows + 7) / 8;
    const int64_t units = rpx * ((m + 15) / 16) * ((dm.k + 15) / 16);
    hipLaunchKernelGGL(k_coupling_tile, dim3((unsigned)(8 * units)), dim3(256), 0, st, dm.k, m, nrows, rpx, rows,
                       dm.adm_ptr, dm.adm_col, S, dm.s_blk, xh, yh, ldh, skip, jpass);
}

// ranks above 64; nj_force: column tiles per work-group (0: as many as the columns fill, fewer
// where the rows do not fill the chip; rank 125, 64 columns: 381 rows 527 us with 4 tiles, 434
// with 2, 745 rows 850 and 820)
inline void launch_coupling_rows(const DevMat &dm, int64_t m, const double *xh, double *yh, int64_t ldh,
                                 hipStream_t st, Skip skip, int nj_force) {
    if (dm.C <= 0) return;
    const double *S = (const double *)dm.S;
    if (!nj_force && coupling_in_tiles(dm.k, m, dm.C))
        return launch_coupling_tile(dm, m, S, xh, yh, ldh, st, skip, dm.C, dm.cpl_order, 0);
    const int64_t groups = dm.C * (int64_t)((dm.k + 63) / 64);
    int nj = nj_force ? nj_force : (int)std::min<int64_t>(4, (m + 15) / 16);
    if (!nj_force && nj > 2 && groups * ((m + 16 * nj - 1) / (16 * nj)) < 1000) nj = 2;
    if (!nj_force && nj == 2 && groups * ((m + 31) / 32) < 600) nj = 1;
    const int32_t rpx = (dm.C + 7) / 8;
    const int64_t parts = ((m + 16 * nj - 1) / (16 * nj)) * ((dm.k + 63) / 64);
    auto go = [&](auto NJc) {
        hipLaunchKernelGGL((k_coupling_rows<decltype(NJc)::value>), dim3((unsigned)(8 * rpx * parts)), dim3(256), 0, st,
                           dm.k, m, dm.C, rpx, dm.cpl_order, dm.adm_ptr, dm.adm_col, S, dm.s_blk, xh, yh, ldh, skip);
    };
    switch (nj) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;
    }
}

}  // namespace h2x
