// Matrix-core (MFMA) coupling kernel for the FP64 operator of rank 64 (smaller ranks in
// coupling_small.hpp, larger ones and few rows in coupling_rows.hpp):
//   y_t = sum_{(t,s) in C_t, admissible} S_b x_s     for every row cluster t.
//
// One work-group (4 waves) owns one row cluster t and a slab of up to 64
// columns; wave w owns rows 16w..16w+15 of y_t.  For each block of the list,
// the work-group stages x_s (64 x 16*NJ) in LDS (double-buffered, next block
// loaded while the current one is multiplied) and each wave streams its
// 16 x 64 slice of S_b straight from HBM into registers (one 16-byte load per
// lane per pair of k-steps; S is stored in that operand order, see s_index),
// also one block ahead.  v_mfma_f64_16x16x4f64 accumulates in registers; y_t
// is written once.  No atomics: each row cluster has exactly one owner.
//
// Work-groups are mapped to rows so that each XCD (work-groups are dealt to
// the 8 XCDs round-robin) gets one contiguous eighth of the rows in tree
// order: neighbouring row clusters share most column clusters, so their x_s
// reads hit the XCD's L2.  Within an eighth, longer lists go first.
#pragma once

#include <algorithm>
#include <type_traits>

#include "coupling_rows.hpp"
#include "coupling_small.hpp"
#include "device.hpp"

namespace h2x {

constexpr int kMfmaK = 64;

// doubles of one x_s buffer (see coupling64)
template <int NJ>
constexpr int kCouplingX = NJ > 2 ? 16 * NJ * (kMfmaK + 2) : kMfmaK * (16 * NJ + 1);

// one row cluster t and the 16 NJ columns from j0 on (mc of them exist)
template <int NJ>
__device__ inline void coupling64(int32_t t, int64_t j0, int mc, const int64_t *__restrict__ adm_ptr,
                                  const int32_t *__restrict__ adm_col, const double *__restrict__ S,
                                  const double *__restrict__ xh, double *__restrict__ yh, int64_t ldh, int jpass,
                                  double (*xs)[kCouplingX<NJ>]) {
    constexpr int MC = 16 * NJ;   // columns per work-group
    constexpr int LDX = MC + 1;   // padded LDS row
    // 48 and 64 columns (TR): x_s transposed in LDS (column c is LDS row c, pitch 66 doubles) with the
    // rows of each group of eight in the order of the S operand pairs (row 8 a + 4 h + l at
    // position 8 a + 2 l + h), so one 16-byte read gives a lane the operands of both k-steps of
    // a pair; narrower slabs keep the row-major tile, which measured faster there
    constexpr bool TR = NJ > 2;
    constexpr int LDT = kMfmaK + 2;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const int64_t b0 = adm_ptr[t], b1 = adm_ptr[t + 1];

    dbl4 acc[NJ];
#pragma unroll
    for (int J = 0; J < NJ; ++J) acc[J] = dbl4{0.0, 0.0, 0.0, 0.0};

    if (b1 > b0) {
        // x_s staging, XPT entries per thread.  TR: column `lane` (lanes past MC idle), rows
        // 16 w + u, at scalar addresses and one 32-bit offset (64-bit addresses per entry held
        // twice the registers: 48 columns 0.669 -> 0.587 ms, 64 columns 0.762 -> 0.733 ms at
        // n = 65536); else column tid % MC, rows tid / MC + (256 / MC) u
        constexpr int XPT = TR ? 16 : 4 * NJ;
        const int xc = TR ? lane : tid % MC, xr = 16 * w;
        const bool xin = xc < mc;  // columns past mc re-read column 0 and are zeroed when stored
        // jpass: column c takes its partner c ^ 1 (J x = (-im, re) per complex column)
        const uint32_t off = (uint32_t)((xin ? xc : 0) ^ jpass);
        const bool neg = jpass & ~xc & 1;
        double xv[XPT];
        auto load_x = [&](int32_t s) {
            const double *src = xh + (int64_t)s * kMfmaK * ldh + j0;
#pragma unroll
            for (int u = 0; u < XPT; ++u) {
                if constexpr (TR)
                    xv[u] = (src + (xr + u) * ldh)[off];
                else
                    xv[u] = src[(int64_t)((tid + 256 * u) / MC) * ldh + off];
            }
        };
        typedef double dbl2 __attribute__((ext_vector_type(2)));
        auto store_x = [&](int buf) {
            if constexpr (TR) {
                if (MC < 64 && xc >= MC) return;
                double *dst = &xs[buf][xc * LDT + xr];
#pragma unroll
                for (int a8 = 0; a8 < XPT / 8; ++a8)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const double v0 = neg ? -xv[8 * a8 + l] : xv[8 * a8 + l];
                        const double v1 = neg ? -xv[8 * a8 + 4 + l] : xv[8 * a8 + 4 + l];
                        *(dbl2 *)(dst + 8 * a8 + 2 * l) = xin ? dbl2{v0, v1} : dbl2{0.0, 0.0};
                    }
            } else {
#pragma unroll
                for (int u = 0; u < XPT; ++u) {
                    const double v = neg ? -xv[u] : xv[u];
                    xs[buf][((tid + 256 * u) / MC) * LDX + xc] = xin ? v : 0.0;
                }
            }
        };
        dbl2 sa[8], sn[8];
        auto load_s = [&](int64_t b, dbl2 *dst) {
            // S_b (32 KB) through a buffer resource: streaming loads at 32-bit offsets
            const __amdgpu_buffer_rsrc_t rs = buf_rsrc(S + b * kMfmaK * kMfmaK, kMfmaK * kMfmaK * 8);
#pragma unroll
            for (int kk2 = 0; kk2 < 8; ++kk2)
                dst[kk2] = __builtin_bit_cast(dbl2, buf_ld16<kBufNT>(rs, 16u * (w * 8 * 64 + kk2 * 64 + lane)));
        };

        // the same order of products per accumulator in both layouts
        auto multiply = [&](int buf) {
            const double *xb = xs[buf];
#pragma unroll
            for (int kk2 = 0; kk2 < 8; ++kk2) {
                if constexpr (TR) {
                    dbl2 bq[NJ];  // rows 8 kk2 + lq and 8 kk2 + 4 + lq of column 16 J + lr
#pragma unroll
                    for (int J = 0; J < NJ; ++J) bq[J] = *(const dbl2 *)(xb + (16 * J + lr) * LDT + 8 * kk2 + 2 * lq);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const double a = h ? sa[kk2].y : sa[kk2].x;
#pragma unroll
                        for (int J = 0; J < NJ; ++J)
                            acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, h ? bq[J].y : bq[J].x, acc[J], 0, 0, 0);
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const double a = h ? sa[kk2].y : sa[kk2].x;
                        const int krow = 4 * (2 * kk2 + h) + lq;
#pragma unroll
                        for (int J = 0; J < NJ; ++J) {
                            const double bv = xb[krow * LDX + 16 * J + lr];
                            acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv, acc[J], 0, 0, 0);
                        }
                    }
                }
            }
        };

        // the list in four consecutive parts whose sums are added in order, as in every coupling
        // form of this operator (the tile form gives a part to each wave): the same bits from each
        const int quarter = (int)((b1 - b0 + 3) / 4);
        dbl4 sum[NJ];
#pragma unroll
        for (int J = 0; J < NJ; ++J) sum[J] = dbl4{0.0, 0.0, 0.0, 0.0};
        load_x(adm_col[b0]);
        load_s(b0, sa);
        store_x(0);
        __syncthreads();
        // every load of the loop is unconditional (bounds handled by clamped addresses and
        // selects) and the last block is peeled off, so the compiler's wait counters are
        // exact: the MFMAs wait only for the current block, never for the prefetch
        int left = quarter;
        // the end of a part (rarely taken, kept out of line; nested loops or selects cost the 32-column
        // form 15 %): after the products, or at 32 columns behind the barrier, as a branch between
        // products and stores makes the compiler issue that form's loads late (n = 65536, 32 columns
        // 0.494 -> 0.483 ms; behind the barrier 48 columns on a cube 1.30 -> 1.41 ms)
        auto flush = [&]() {
            if (__builtin_expect(--left == 0, 0)) {
                left = quarter;
#pragma unroll
                for (int J = 0; J < NJ; ++J) {
                    sum[J] += acc[J];
                    acc[J] = dbl4{0.0, 0.0, 0.0, 0.0};
                }
            }
        };
        for (int64_t b = b0; b + 1 < b1; ++b) {
            const int buf = (int)((b - b0) & 1);
            load_x(adm_col[b + 1]);
            load_s(b + 1, sn);
            multiply(buf);
            if constexpr (NJ != 2) flush();
            store_x(buf ^ 1);
#pragma unroll
            for (int kk2 = 0; kk2 < 8; ++kk2) sa[kk2] = sn[kk2];
            __syncthreads();
            if constexpr (NJ == 2) flush();
        }
        multiply((int)((b1 - 1 - b0) & 1));
#pragma unroll
        for (int J = 0; J < NJ; ++J) acc[J] = sum[J] + acc[J];
    }
    // D layout of the 16x16x4 f64 MFMA: lane l, register r -> row l / 16 + 4 r, column l % 16
#pragma unroll
    for (int J = 0; J < NJ; ++J) {
        const int col = 16 * J + lr;
        if (col < mc) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * w + lq + 4 * r;
                double *y = &yh[((int64_t)t * kMfmaK + row) * ldh + j0 + col];
                *y = jpass ? *y + acc[J][r] : acc[J][r];  // the second pass adds
            }
        }
    }
}

// NJL: column tiles of the last slab (a slab of 64 columns for the 36 that remain of 100 would
// multiply 28 columns of padding; n = 65536, 80 columns: 1.476 -> 1.380 ms, 100 columns: 1.507 -> 1.420)
template <int NJ, int NJL>
__global__ __launch_bounds__(256) void k_coupling_mfma_f64(int64_t m, int32_t C, int32_t rows_per_xcd,
                                                           const int32_t *__restrict__ order,
                                                           const int64_t *__restrict__ adm_ptr,
                                                           const int32_t *__restrict__ adm_col,
                                                           const double *__restrict__ S,
                                                           const double *__restrict__ xh, double *__restrict__ yh,
                                                           int64_t ldh, Skip skip, int jpass) {
    constexpr int MC = 16 * NJ;
    __shared__ __align__(16) double xs[2][kCouplingX<NJ>];
    // the column slabs of one row cluster are consecutive work-groups of one XCD, so S_b
    // comes from HBM once and from that XCD's L2 for the other slabs
    const int nslab = (int)((m + MC - 1) / MC), qx = blockIdx.x >> 3;
    const int slot = (blockIdx.x & 7) * rows_per_xcd + qx / nslab;
    if (slot >= C) return;
    const int32_t t = order[slot];
    if (skip(t)) return;
    const int64_t j0 = (int64_t)(qx % nslab) * MC;
    if constexpr (NJL < NJ) {
        static_assert(kCouplingX<NJL> <= kCouplingX<NJ>, "the last slab's buffers fit");
        if (j0 + MC > m)
            return coupling64<NJL>(t, j0, (int)(m - j0), adm_ptr, adm_col, S, xh, yh, ldh, jpass,
                                   (double(*)[kCouplingX<NJL>])xs);
    }
    coupling64<NJ>(t, j0, (int)min<int64_t>(MC, m - j0), adm_ptr, adm_col, S, xh, yh, ldh, jpass, xs);
}

// The coupling stage of the ranks up to 64 (dm.mc).
inline void launch_coupling(const DevMat &dm, int64_t m, const double *xh, double *yh, int64_t ldh, hipStream_t st,
                            Skip skip, int nj_force, int jpass = 0, int32_t nrows = -1, const int32_t *rows = nullptr,
                            size_t keep_lds = 0) {
    // all rows in cpl_order, or the part (nrows, rows) of them
    const int32_t C = rows ? nrows : dm.C;
    const int32_t *order = rows ? rows : dm.cpl_order;
    if (C <= 0) return;
    // column tiles per work-group: as many as the columns fill, fewer where the rows alone do not
    // fill the chip (rank 64, sphere: 375 rows, 64 columns: 4 tiles 151, 2 tiles 116 us; 745 rows:
    // 198 and 214 us; 32 columns, 193 rows: 82 and 67 us); the bits do not depend on it
    int nj = nj_force ? nj_force : (int)std::min<int64_t>(4, (m + 15) / 16);
    if (!nj_force && dm.k == kMfmaK) {
        if (nj > 2 && C * ((m + 16 * nj - 1) / (16 * nj)) < 720) nj = 2;
        if (nj == 2 && C * ((m + 31) / 32) < 600) nj = 1;
    }
    const int mcols = 16 * nj;
    const int32_t rpx = (C + 7) / 8;
    const dim3 grid((unsigned)(8 * rpx * ((m + mcols - 1) / mcols)));
    // jpass (complex operator): the imaginary plane of S on J x-hat, added to y-hat
    const double *S = (const double *)dm.S + (jpass ? dm.s_plane : 0);
    if (dm.k <= 32) {
        launch_coupling_small(dm, m, S, xh, yh, ldh, st, skip, nj_force, C, order, jpass);
        return;
    }
    if (!nj_force && !keep_lds && coupling_in_tiles(dm.k, m, C)) {
        launch_coupling_tile(dm, m, S, xh, yh, ldh, st, skip, C, order, jpass);
        return;
    }
    // keep_lds > 0: each work-group also takes unused dynamic LDS, so that a CU holds at
    // most two of them and keep_lds bytes stay free for a work-group of another launch
    // (the work-groups of a long launch must not take every slot of the chip)
    auto dyn_lds = [&](const void *fn) -> size_t {
        if (!keep_lds) return 0;
        hipFuncAttributes a{};
        int dev = 0, per_cu = 0;
        if (hipFuncGetAttributes(&a, fn) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
                hipSuccess || (size_t)per_cu <= keep_lds)
            return 0;
        const size_t target = (((size_t)per_cu - keep_lds) / 2) & ~(size_t)255;
        return target > a.sharedSizeBytes ? target - a.sharedSizeBytes : 0;
    };
    auto go = [&](auto NJc, auto NJLc) {
        constexpr int NJ = decltype(NJc)::value, NJL = decltype(NJLc)::value;
        const size_t dyn = dyn_lds((const void *)k_coupling_mfma_f64<NJ, NJL>);
        hipLaunchKernelGGL((k_coupling_mfma_f64<NJ, NJL>), grid, dim3(256), dyn, st, m, C, rpx, order, dm.adm_ptr,
                           dm.adm_col, S, xh, yh, ldh, skip, jpass);
    };
    auto one = std::integral_constant<int, 1>{};
    auto two = std::integral_constant<int, 2>{};
    auto three = std::integral_constant<int, 3>{};
    auto four = std::integral_constant<int, 4>{};
    switch (nj) {
        case 1: go(one, one); break;
        case 2: go(two, two); break;
        case 3: go(three, three); break;
        default: {
            const int64_t rest = m % 64;  // columns of the last slab
            if (m < 64 || rest == 0 || rest > 48) go(four, four);
            else if (rest > 32) go(four, three);
            else if (rest > 16) go(four, two);
            else go(four, one);
        }
    }
}

}  // namespace h2x
