// Leaf stage of the FP32 / BF16 operators as one contraction per leaf (FP32 matrix cores):
//
//   Y|_t = beta Y|_t + alpha (V_t y_t + sum_{(t,s) near} N_ts X|_s)
//
// the organisation of the FP64 form in leaf_cat.hpp with v_mfma_f32_16x16x4f32: the
// transposed near blocks of a leaf (FP32, rows padded to an even length) and its transposed
// basis (FP32 or BF16) form one matrix of sum |s| + k rows, contracted in rounds of 16 rows
// against rows of the FP32 tree-ordered copy of X (through the per-leaf table of near rows in
// LDS) or of y_t; FP32 sums.  With a BF16 basis, y_t is rounded to BF16 where it meets V_t
// (both factors of a product in the storage type).  Only the end of each segment is padded (to
// 16 rows) and the rows of the leaf come in 16-row tiles.
//
// Work-group: two or four waves for one (leaf, slab of 16 NC columns).  Two waves each take every
// second round for all row tiles of a 64-row chunk and all column tiles, so every operand is loaded
// once per work-group; four waves split chunks above 32 rows into two row groups or, for three row
// tiles and an even NC, two column halves (each loads one operand for itself), so that few leaves
// still fill the chip.  The sums are the same bit for bit.  Bound by the FP32 matrix cores and the
// loads that feed them.  Slabs of 32 or 64 columns spent up to a quarter of the products on padding
// and row groups 22 GB of cache traffic where 13 do: 45 columns, n = 99991, BF16 basis, leaf stage
// 1029 -> 790 us; 64 columns, n = 262144, FP32 2330 -> 2150 us.  Above four tiles per wave the
// registers allow two waves per SIMD and one round of loads ahead (two rounds ahead spill: 5 x
// slower, half rounds three ahead are 1 % slower); up to four tiles of a chunk above 32 rows two
// rounds fly (leaves of up to 100 points, 32 columns, BF16: leaf stage 335 -> 315 us).  The row
// table and the partial tiles take the same LDS (beside each other: + 8 % of a product with tables
// of 30 KB).
//
// Lane layout of v_mfma_f32_16x16x4f32 (A: 16 x 4, B: 4 x 16, D: 16 x 16): lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D rows 4 (l / 16) + q, column l % 16 (q = 0..3).
// Here A = X^T and B = N^T: a lane loads two neighbouring columns (rows) with one 8-byte load,
// which feed an "even" and an "odd" tile; an odd last tile is loaded by 4 bytes per lane.
#pragma once

#include "leaf_cat.hpp"
#include "leaf_lp.hpp"

namespace h2x {
namespace lp {

template <int NC, int NT>
struct CatRoundLp {
    flt2 a[NC / 2 + 1][4];  // [column pair p][k-step u]: columns 32p + 2 (l % 16) + {0, 1}
    float c[4];             // [k-step u], NC odd: column 16 (NC - 1) + l % 16
    flt2 b[NT / 2 + 1][4];  // [row pair q][k-step u]: rows 32q + 2 (l % 16) + {0, 1}
    float d[4];             // [k-step u], NT odd: row 16 (NT - 1) + l % 16
};

__device__ inline float ld1(const float *p) { return *p; }
__device__ inline float ld1(const bf16_t *p) { return __builtin_bit_cast(float, (uint32_t)p->b << 16); }

struct LeafCatLpArgs {
    int k;
    int64_t m;
    int32_t L;
    const int32_t *order;  // launch order of the leaves (leaf indices)
    const int32_t *leaves, *first, *size;
    const int64_t *perm;
    const void *Vt;  // transposed leaf bases, FP32 or BF16
    const int64_t *vt_off;
    const float *yh;
    int64_t ldh;
    const int64_t *near_ptr;
    const int32_t *near_col;
    const int64_t *near_off;
    const float *Nt, *Xt;
    int64_t ldxt;
    double alpha, beta;
    double *Y;
    int64_t ldy;
    int tree_order;
    Skip skip;
};

// NT row tiles from row i0 on (ic of these rows present) and NC column tiles.  The rounds are summed
// in G groups (group r % G: two where the chunk has three or four row tiles, four below); of the GW
// waves of these rows, wave g takes the groups g, g + GW, .. in turn.  The groups' partial tiles
// are added in LDS in order (red: their first row).
template <int NC, int NT, int G, int GW, int LDR, typename TV>
__device__ inline void leaf_cat_lp_chunk(const LeafCatLpArgs &a, int g, int lr, int lq, int32_t t, const float *nb,
                                         const TV *vb, int32_t rn, int64_t nt2, int i0, int ic, int64_t j0, int xc,
                                         const int32_t *xrow, float *red) {
    constexpr int NA = G / GW, NPR = NC / 2;
    const int k = a.k;
    const int RN = (rn + 15) >> 4, RT = RN + ((k + 15) >> 4);
    // (row lengths are even: a pair stays inside its row)
    uint32_t row[NT / 2 + 1];
#pragma unroll
    for (int q = 0; q < NT / 2; ++q) row[q] = (uint32_t)(i0 + min(32 * q + 2 * lr, (ic - 1) & ~1));
    const uint32_t rs = (uint32_t)(i0 + min(16 * (NT - 1) + lr, ic - 1));
    uint32_t cp[NPR + 1];
#pragma unroll
    for (int p = 0; p < NPR; ++p) cp[p] = (uint32_t)min(32 * p + 2 * lr, xc);
    const uint32_t cs = (uint32_t)min(16 * (NC - 1) + lr, xc + 1);

    flt4v acc[NA][NC][NT];
#pragma unroll
    for (int x = 0; x < NA; ++x)
#pragma unroll
        for (int J = 0; J < NC; ++J)
#pragma unroll
            for (int I = 0; I < NT; ++I) acc[x][J][I] = flt4v{0.f, 0.f, 0.f, 0.f};

    // round r -> registers; both branches issue the same number of loads from clamped in-range
    // addresses, so the wait counts stay exact.  The near-field operands come through buffer
    // resources (32-bit byte offsets; the host takes this form only while X is below 4 GiB).
    auto load = [&](int r, CatRoundLp<NC, NT> &R) {
        if (r < RN) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cc = min(16 * r + 4 * u + lq, rn - 1);
                const __amdgpu_buffer_rsrc_t rx = buf_rsrc(a.Xt + j0, 0xFFFFFFFFu), rb = buf_rsrc(nb, 0xFFFFFFFFu);
                const uint32_t xo = (uint32_t)(xrow[cc] * a.ldxt), bo = (uint32_t)(cc * nt2);
#pragma unroll
                for (int p = 0; p < NPR; ++p) R.a[p][u] = __builtin_bit_cast(flt2, buf_ld8<0>(rx, 4u * (xo + cp[p])));
                if (NC & 1) R.c[u] = buf_ld4f<0>(rx, 4u * (xo + cs));
#pragma unroll
                for (int q = 0; q < NT / 2; ++q)
                    R.b[q][u] = __builtin_bit_cast(flt2, buf_ld8<0>(rb, 4u * (bo + row[q])));
                if (NT & 1) R.d[u] = buf_ld4f<0>(rb, 4u * (bo + rs));
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cc = min(16 * (r - RN) + 4 * u + lq, k - 1);
                const float *ar = a.yh + ((int64_t)t * k + cc) * a.ldh + j0;
#pragma unroll
                for (int p = 0; p < NPR; ++p) R.a[p][u] = ld2(ar + cp[p]);
                if (NC & 1) R.c[u] = ar[cs];
#pragma unroll
                for (int q = 0; q < NT / 2; ++q) R.b[q][u] = ld2(vb + (int64_t)cc * nt2 + row[q]);
                if (NT & 1) R.d[u] = ld1(vb + (int64_t)cc * nt2 + rs);
            }
        }
    };
    // the products of round r; rows past its segment are zeroed here
    auto multiply = [&](int r, const CatRoundLp<NC, NT> &R, flt4v(&ac)[NC][NT]) {
        const bool basis = r >= RN;
        const int rem = basis ? k - 16 * (r - RN) : rn - 16 * r;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = 4 * u + lq < rem;
#pragma unroll
            for (int J = 0; J < NC; ++J) {
                float v = ((NC & 1) && J == NC - 1) ? R.c[u] : R.a[J >> 1][u][J & 1];
                v = ok ? v : 0.f;
                // (not in the FP32 kernel: the branches of a rounding split a round's products up)
                if constexpr (std::is_same<TV, bf16_t>::value)
                    if (basis) v = round_bf16(v);
#pragma unroll
                for (int I = 0; I < NT; ++I)
                    ac[J][I] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        v, ((NT & 1) && I == NT - 1) ? R.d[u] : R.b[I >> 1][u][I & 1], ac[J][I], 0, 0, 0);
            }
        }
    };

    if (g < RT) {
        const int last = g + ((RT - 1 - g) / GW) * GW;  // the wave's last round
        int r = g;
        if constexpr (NA == 1 && G == 2 && NC * NT <= 4) {
            // three register sets in turn; a set is loaded two rounds ahead of its use (a round past
            // the last re-reads that one, which the cache serves)
            CatRoundLp<NC, NT> s0, s1, s2;
            load(r, s0);
            load(min(r + GW, last), s1);
            for (;;) {
                load(min(r + 2 * GW, last), s2);
                multiply(r, s0, acc[0]);
                if ((r += GW) > last) break;
                load(min(r + 2 * GW, last), s0);
                multiply(r, s1, acc[0]);
                if ((r += GW) > last) break;
                load(min(r + 2 * GW, last), s1);
                multiply(r, s2, acc[0]);
                if ((r += GW) > last) break;
            }
        } else {  // two sets, one round ahead
            CatRoundLp<NC, NT> s0, s1;
            load(r, s0);
            for (;;) {
                load(min(r + GW, last), s1);
                multiply(r, s0, acc[0]);
                if ((r += GW) > last) break;
                load(min(r + GW, last), s0);
                multiply(r, s1, acc[NA - 1]);
                if ((r += GW) > last) break;
            }
        }
    }
    __syncthreads();  // the row table was read for the last time: its LDS takes the partial tiles
    // Lane l, register q of a pair tile J -> column 32 (J / 2) + 2 (4 (l / 16) + q) + J % 2, of a
    // single last tile -> column 16 (NC - 1) + 4 (l / 16) + q; rows as in the loads.
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
        if (g == gg % GW)
#pragma unroll
            for (int J = 0; J < NC; ++J)
#pragma unroll
                for (int I = 0; I < NT; ++I) {
                    const int row = ((NT & 1) && I == NT - 1) ? 16 * I + lr : 32 * (I >> 1) + 2 * lr + (I & 1);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col = ((NC & 1) && J == NC - 1) ? 16 * J + 4 * lq + q
                                                                  : 32 * (J >> 1) + 2 * (4 * lq + q) + (J & 1);
                        float *cell = &red[row * LDR + col];
                        const float v = acc[gg / GW][J][I][q];
                        *cell = (gg == 0) ? v : *cell + v;
                    }
                }
        __syncthreads();
    }
}

// one (leaf, column slab) per work-group, mapped to XCDs as in the FP64 form (slot & 7 is the
// XCD, whose leaves form one contiguous eighth of the launch order; the slabs of one leaf are
// consecutive slots of one XCD).  Dynamic LDS: the near-row table, then the partial tiles.
// ROWS: the largest leaf, 32, 64 or 128 for any.  64: the lane's number is opaque in each chunk, as the
// offsets of every form would else be held across the table's barriers (32 columns: 139 registers,
// three waves per SIMD; 121, four; cube 60000, BF16 786 -> 772 us per product; larger leaves, two
// chunks each, are faster without: sphere 79040, leaves of 80, FP32 526 / 536).
template <int NC, int NW, int ROWS, typename TV>
__global__ __launch_bounds__(64 * NW, 2) void k_leaf_cat_lp(LeafCatLpArgs a) {
    constexpr int MC = 16 * NC, LDR = MC + 1;
    extern __shared__ float red[];
    int32_t *xrow = (int32_t *)red;
    const int64_t slot = blockIdx.x;
    const int32_t per_xcd = (a.L + 7) / 8;
    const int nslab = (int)((a.m + MC - 1) / MC);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t qx = slot >> 3;
    const int32_t pos = (int32_t)((slot & 7) * per_xcd + qx / nslab);
    if (pos >= a.L) return;
    const int32_t l = a.order[pos];
    const int32_t t = a.leaves[l];
    if (a.skip(t)) return;
    const int nt = a.size[t];
    const int64_t nt2 = pad_rows(nt), r0 = a.first[t];
    const int64_t j0 = (qx % nslab) * MC;
    const int mc = (int)min<int64_t>(MC, a.m - j0);
    const int64_t q0 = a.near_ptr[l];
    const int nnear = (int)(a.near_ptr[l + 1] - q0);
    const float *nb = nnear > 0 ? a.Nt + a.near_off[q0] : a.Nt;
    const TV *vb = (const TV *)a.Vt + a.vt_off[l];
    const int xc = (mc - 1) & ~1;  // last even column offset of the slab
    for (int i0 = 0; i0 < nt; i0 += 64) {
        const int32_t rn =
            nnear > 0 ? mfma::cat_build_rows(xrow, q0, nnear, nt2, a.near_col, a.near_off, a.first, a.size, threadIdx.x)
                      : 0;
        const int ic = min(64, nt - i0);
        int lane = threadIdx.x & 63;
        if (ROWS == 64) asm volatile("" : "+v"(lane));
        const int lr = lane & 15, lq = lane >> 4;
        if (ic <= 16)
            leaf_cat_lp_chunk<NC, 1, 4, NW, LDR>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        else if (ROWS <= 32 || ic <= 32)
            leaf_cat_lp_chunk<NC, 2, 4, NW, LDR>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        else if constexpr (ROWS > 32) {
            if (NW == 4 && NC % 2 == 0 && ic <= 48 && mc > 8 * NC) {
                // two waves per column half: equal work for three row tiles
                constexpr int HC = NC > 1 ? NC / 2 : 1;
                const int ch = 16 * HC * (w >> 1);
                leaf_cat_lp_chunk<HC, 3, 2, 2, LDR>(a, w & 1, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0 + ch, xc - ch,
                                                    xrow, red + ch);
            } else if (NW == 4)  // two waves per 32 rows
                leaf_cat_lp_chunk<NC, 2, 2, 2, LDR>(a, w & 1, lr, lq, t, nb, vb, rn, nt2, i0 + 32 * (w >> 1),
                                                    w < 2 ? 32 : ic - 32, j0, xc, xrow, red + (w >> 1) * 32 * LDR);
            else if (ic <= 48)
                leaf_cat_lp_chunk<NC, 3, 2, 2, LDR>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
            else
                leaf_cat_lp_chunk<NC, 4, 2, 2, LDR>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        }
        for (int x = threadIdx.x; x < ic * MC; x += 64 * NW) {
            const int i = x / MC, j = x - i * MC;
            if (j < mc) {
                int64_t row = r0 + i0 + i;
                if (!a.tree_order) row = a.perm[row];
                double *y = &a.Y[row * a.ldy + j0 + j];
                const double v = a.alpha * (double)red[i * LDR + j];
                *y = (a.beta == 0.0) ? v : a.beta * *y + v;
            }
        }
        __syncthreads();
    }
}

}  // namespace lp
}  // namespace h2x
