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

#include "device.hpp"
#include "matmul_mfma.hpp"

namespace h2x {

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
        int c = 0;
        int64_t b = b0;
        load(b0, 0, sa);
        store(0, 0);
        __syncthreads();
        int buf = 0;
        for (;;) {
            const int cn = c + 1 < nch ? c + 1 : 0;
            const int64_t bn = cn ? b : b + 1;
            if (bn >= b1) break;
            load(bn, cn, sn);
            multiply(buf, c);
            store(buf ^ 1, cn);
#pragma unroll
            for (int q = 0; q < 8; ++q) sa[q] = sn[q];
            __syncthreads();
            b = bn;
            c = cn;
            buf ^= 1;
        }
        multiply(buf, c);
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

inline void launch_coupling_rows(const DevMat &dm, int64_t m, const double *xh, double *yh, int64_t ldh,
                                 hipStream_t st, Skip skip) {
    if (dm.C <= 0) return;
    const int nj = (int)std::min<int64_t>(4, (m + 15) / 16);
    const int32_t rpx = (dm.C + 7) / 8;
    const int64_t parts = ((m + 16 * nj - 1) / (16 * nj)) * ((dm.k + 63) / 64);
    const dim3 grid((unsigned)(8 * rpx * parts));
    auto go = [&](auto NJc) {
        hipLaunchKernelGGL(k_coupling_rows<decltype(NJc)::value>, grid, dim3(256), 0, st, dm.k, m, dm.C, rpx,
                           dm.cpl_order, dm.adm_ptr, dm.adm_col, (const double *)dm.S, dm.s_blk, xh, yh, ldh, skip);
    };
    switch (nj) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;
    }
}

}  // namespace h2x
