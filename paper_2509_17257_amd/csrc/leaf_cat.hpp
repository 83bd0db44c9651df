// Leaf stage of the FP64 operator as one contraction per leaf (matrix cores).
//
//   Y|_t = beta Y|_t + alpha (V_t y_t + sum_{(t,s) near} N_ts X|_s)
//
// computed in the transposed orientation Y_t^T = [X_s1^T ... X_sq^T y_t^T] [N_ts1^T; ...; N_tsq^T; V_t^T]:
// the near blocks of a leaf are stored transposed one after another with the same row
// length |t| (padded to even), so the near field of leaf t is one matrix of R_t = sum |s|
// rows, and the transposed leaf basis adds k rows.  The contraction runs over these rows in
// rounds of 16 (four 4-long matrix-core steps); the right operand of a row is the row of X
// of its point (a per-leaf table in LDS maps near rows to tree positions) or the row of
// y_t.  Only the end of each segment is padded (to 16 rows), and the rows of the leaf come
// in 16-row tiles, so a leaf of 43 points and 1100 near rows costs 48 x 1104 instead of
// 64 x 1152 terms per column.
//
// Work-group: four waves for one (leaf, slab of 16 NC columns).  Chunks of up to 32 rows of a leaf
// are one row group (of one tile up to 16 rows) and the waves split the rounds (wave w takes
// rounds w, w + 4, ...); larger chunks are two row groups of two tiles, or, for three row tiles
// and an even NC, two column halves, each split over two waves (two tiles throughout, present or
// not: leaves of 16, 64 columns, cube of 65536 leaf stage 462 against 319 us; leaves of up to 75, 32
// columns 458 against 424).  With two waves per work-group each takes every second round for all
// rows.  The partial tiles are added in LDS in wave order (a fixed order, the same for every form:
// the result is reproducible and does not depend on the form).  Complex operators: every wave
// all rows of every fourth round.  One or two further rounds of
// loads stay in flight behind the matrix-core work of the current one; every load is issued
// unconditionally from a clamped in-range address (a round past the wave's last re-reads that
// round, which the cache serves) so that the compiler's wait counts stay exact, and rows past
// a segment are zeroed where they are used.  A complex operator's near field is two sets of
// rounds over the same rows, its real plane on X and its imaginary plane on J X.
//
// Bound by HBM for few columns and by the matrix cores from 64 on; what is lost is latency: the
// chain of tables before a leaf's first load, and too few loads in flight.  Slabs of 16-column
// tiles (32 or 64 columns before), pairs of rows by one 16-byte load, the row table in the LDS
// of the partial tiles (one more work-group per CU), and the complex operator in this form:
// product at n = 65536, m = 1 633 -> 594 us; n = 32768, leaf 128, m = 16 720 -> 671 us; complex
// n = 32768, 8 columns 715 -> 629 us.  Three register sets at two column tiles spill.
//
// Lane layout of v_mfma_f64_16x16x4f64 (A: 16 x 4, B: 4 x 16, D: 16 x 16): lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D rows l / 16 + 4 r, column l % 16 (r = 0..3).
// Here A = X^T (M over columns of X), B = N^T (N over rows of the leaf): a lane loads two
// neighbouring columns (rows) with one 16-byte load, which feed an "even" and an "odd" tile; an
// odd last tile is loaded by 8 bytes per lane.
#pragma once

#include <type_traits>

#include "device.hpp"
#include "stages_mfma.hpp"

namespace h2x {
namespace mfma {

typedef double dbl4c __attribute__((ext_vector_type(4)));
typedef double dbl2c __attribute__((ext_vector_type(2)));

// registers of one round of a wave (NC column tiles, NT row tiles)
template <int NC, int NT>
struct CatRound {
    dbl2c a[NC / 2 + 1][4];  // [column pair p][k-step u]: columns 32p + 2 (l % 16) + {0, 1}
    double c[4];             // [k-step u], NC odd: column 16 (NC - 1) + l % 16
    dbl2c b[NT / 2 + 1][4];  // [row pair q][k-step u]: rows 32q + 2 (l % 16) + {0, 1}
    double d[4];             // [k-step u], NT odd: row 16 (NT - 1) + l % 16
};

// rows of the near field of one leaf, as a table of tree positions in LDS (built from the
// blocks' offsets: block q starts at near row (off_q - off_q0) / |t|_even)
__device__ inline int32_t cat_build_rows(int32_t *xrow, int64_t q0, int nnear, int64_t nt2,
                                         const int32_t *__restrict__ near_col, const int64_t *__restrict__ near_off,
                                         const int32_t *__restrict__ first, const int32_t *__restrict__ size,
                                         int tid) {
    __shared__ int32_t rn;
    const int64_t base = near_off[q0];
    if (tid == 0) rn = 0;
    __syncthreads();
    for (int x = tid; x < nnear; x += blockDim.x) {
        const int32_t s = near_col[q0 + x];
        const int32_t off = (int32_t)((near_off[q0 + x] - base) / nt2), fs = first[s], ks = size[s];
        for (int c = 0; c < ks; ++c) xrow[off + c] = fs + c;
        if (x == nnear - 1) rn = off + ks;
    }
    __syncthreads();
    return rn;
}

// the leaf stage's arguments (one struct, shared by the kernels that run leaf work)
struct LeafCatArgs {
    int k;
    int64_t m;
    int32_t L;
    const int32_t *order;  // launch order of the leaves (leaf indices)
    const int32_t *leaves, *first, *size;
    const int64_t *perm;
    const double *Vt;
    const int64_t *vt_off;
    const double *yh;
    int64_t ldh;
    const int64_t *near_ptr;
    const int32_t *near_col;
    const int64_t *near_off;
    const double *Nt, *Xt;
    int64_t ldxt;
    double alpha, beta;
    double *Y;
    int64_t ldy;
    int tree_order, basis, near;
    Skip skip;
    int64_t n_plane;  // complex operator: offset of the imaginary parts in Nt, else 0
};

// LDS of the leaf work: the near-row table, then the partial tiles of a slab of 16 NC columns
__host__ __device__ constexpr size_t leaf_cat_red_bytes(int NC) { return sizeof(double) * 64 * (16 * NC + 1); }

// NT row tiles from row i0 on (ic of these rows present) and NC column tiles from column j0 on.  The
// rounds are summed in G groups (group r % G: two where the chunk has three or four row tiles, four
// below); of the GW waves of these rows, wave g takes the groups g, g + GW, .. in turn.  The
// groups' partial tiles are added in LDS in order (red: the first cell, rows of LDR).  CPX: the
// near rounds run on two waves for the real plane on X and on two for the imaginary plane on J X
// (column pairs (re, im) -> (-im, re)), so the large diagonal entries meet a quarter of the terms.
template <int NC, int NT, int G, int GW, int LDR, bool CPX>
__device__ inline void leaf_cat_chunk(const LeafCatArgs &a, int g, int lr, int lq, int32_t t, const double *nb,
                                      const double *vb, int32_t rn, int64_t nt2, int i0, int ic, int64_t j0, int xc,
                                      const int32_t *xrow, double *red) {
    constexpr int NA = G / GW, NPR = NC / 2;
    const int k = a.k;
    const int RN = (rn + 15) >> 4, RI = CPX ? 4 * ((RN + 1) >> 1) : RN, RT = RI + (a.basis ? (k + 15) >> 4 : 0);
    // (row lengths are even: a pair stays inside its row; the blocks of a leaf are below 4 GiB, as
    // their table fits in LDS)
    const uint32_t len = (uint32_t)nt2;
    uint32_t row[NT / 2 + 1];
#pragma unroll
    for (int q = 0; q < NT / 2; ++q) row[q] = (uint32_t)(i0 + min(32 * q + 2 * lr, (ic - 1) & ~1));
    const uint32_t rs = (uint32_t)(i0 + min(16 * (NT - 1) + lr, ic - 1));
    uint32_t cp[NPR + 1];
#pragma unroll
    for (int p = 0; p < NPR; ++p) cp[p] = (uint32_t)min(32 * p + 2 * lr, xc);
    const uint32_t cs = (uint32_t)min(16 * (NC - 1) + lr, xc + 1);

    dbl4c acc[NA][NC][NT];
#pragma unroll
    for (int x = 0; x < NA; ++x)
#pragma unroll
        for (int J = 0; J < NC; ++J)
#pragma unroll
            for (int I = 0; I < NT; ++I) acc[x][J][I] = dbl4c{0.0, 0.0, 0.0, 0.0};

    // rows 16 near_round(r).. of the near field: of four rounds of a complex operator the first two
    // are the real plane's, the last two the imaginary plane's
    auto near_round = [](int r) { return CPX ? 2 * (r >> 2) + (r & 1) : r; };
    // round r -> registers, from clamped in-range addresses (X and y_t: 32-bit byte offsets)
    auto load = [&](int r, CatRound<NC, NT> &R) {
        const bool nr = r < RI, im = CPX && nr && (r & 2);
        const double *ab = nr ? a.Xt + j0 : a.yh + (int64_t)t * k * a.ldh + j0;
        const int64_t lda = nr ? a.ldxt : a.ldh;
        const double *bb = nr ? nb + (im ? a.n_plane : 0) : vb;
        const int c0 = 16 * (nr ? near_round(r) : r - RI), lim = nr ? rn : k;
        const uint32_t sw = im ? 1 : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int cc = min(c0 + 4 * u + lq, lim - 1);
            const uint32_t ao = (uint32_t)((nr ? (int64_t)xrow[cc] : (int64_t)cc) * lda);
#pragma unroll
            for (int p = 0; p < NPR; ++p)
                R.a[p][u] = __builtin_bit_cast(dbl2c, buf_ld16<0>(buf_rsrc(ab, 0xFFFFFFFFu), 8u * (ao + cp[p])));
            if (NC & 1)
                R.c[u] = __builtin_bit_cast(double, buf_ld8<0>(buf_rsrc(ab, 0xFFFFFFFFu), 8u * (ao + (cs ^ sw))));
#pragma unroll
            for (int q = 0; q < NT / 2; ++q)
                R.b[q][u] = __builtin_bit_cast(dbl2c, buf_ld16<0>(buf_rsrc(bb, 0xFFFFFFFFu), 8u * (cc * len + row[q])));
            if (NT & 1)
                R.d[u] = __builtin_bit_cast(double, buf_ld8<0>(buf_rsrc(bb, 0xFFFFFFFFu), 8u * (cc * len + rs)));
        }
    };
    // the products of round r; rows past its segment are zeroed here
    auto multiply = [&](int r, const CatRound<NC, NT> &R, dbl4c(&ac)[NC][NT]) {
        const bool im = CPX && r < RI && (r & 2);
        const int rem = r < RI ? rn - 16 * near_round(r) : k - 16 * (r - RI);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = 4 * u + lq < rem;
#pragma unroll
            for (int J = 0; J < NC; ++J) {
                double v;
                if ((NC & 1) && J == NC - 1) {
                    v = R.c[u];
                    if (im && !(lr & 1)) v = -v;
                } else {
                    v = R.a[J >> 1][u][J & 1];
                    if (im) v = (J & 1) ? R.a[J >> 1][u][0] : -R.a[J >> 1][u][1];
                }
                v = ok ? v : 0.0;
#pragma unroll
                for (int I = 0; I < NT; ++I)
                    ac[J][I] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        v, ((NT & 1) && I == NT - 1) ? R.d[u] : R.b[I >> 1][u][I & 1], ac[J][I], 0, 0, 0);
            }
        }
    };

    if (g < RT) {
        const int last = g + ((RT - 1 - g) / GW) * GW;  // the wave's last round
        int r = g;
        if constexpr (NA == 1 && NC * NT <= 2) {
            // three register sets in turn; a set is loaded two rounds ahead of its use (a round past
            // the last re-reads that one, which the cache serves)
            CatRound<NC, NT> s0, s1, s2;
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
            CatRound<NC, NT> s0, s1;
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
    // Lane l, register q of a pair tile J -> column 32 (J / 2) + 2 (l / 16 + 4 q) + J % 2, of a single
    // last tile -> column 16 (NC - 1) + l / 16 + 4 q; rows as in the loads.
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
        if (g == gg % GW)
#pragma unroll
            for (int J = 0; J < NC; ++J)
#pragma unroll
                for (int I = 0; I < NT; ++I) {
                    const int rw = ((NT & 1) && I == NT - 1) ? 16 * I + lr : 32 * (I >> 1) + 2 * lr + (I & 1);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col = ((NC & 1) && J == NC - 1) ? 16 * J + lq + 4 * q
                                                                  : 32 * (J >> 1) + 2 * (lq + 4 * q) + (J & 1);
                        double *cell = &red[rw * LDR + col];
                        const double v = acc[gg / GW][J][I][q];
                        *cell = (gg == 0) ? v : *cell + v;
                    }
                }
        __syncthreads();
    }
}

// columns j0..j0 + 16 NC - 1 of leaf l by NW waves; red: the dynamic LDS
template <int NC, int NW, bool CPX>
__device__ inline void leaf_cat_slab(int32_t l, int64_t j0, const LeafCatArgs &a, double *red, int tid) {
    constexpr int MC = 16 * NC, LDR = MC + 1;
    int32_t *xrow = (int32_t *)red;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int32_t t = a.leaves[l];
    if (a.skip(t)) return;
    const int nt = a.size[t];
    const int64_t nt2 = pad_rows(nt), r0 = a.first[t];
    const int mc = (int)min<int64_t>(MC, a.m - j0);
    const int64_t q0 = a.near_ptr[l];
    const int nnear = a.near ? (int)(a.near_ptr[l + 1] - q0) : 0;
    const double *nb = nnear > 0 ? a.Nt + a.near_off[q0] : a.Nt;
    const double *vb = a.Vt + a.vt_off[l];
    const int xc = (mc - 1) & ~1;  // last even column offset of the slab

    for (int i0 = 0; i0 < nt; i0 += 64) {
        const int32_t rn =
            nnear > 0 ? cat_build_rows(xrow, q0, nnear, nt2, a.near_col, a.near_off, a.first, a.size, tid) : 0;
        const int ic = min(64, nt - i0);
        if constexpr (CPX) {  // four groups: the sums are twice as long
            if (ic <= 32)
                leaf_cat_chunk<NC, 2, 4, 4, LDR, true>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
            else if (ic <= 48)
                leaf_cat_chunk<NC, 3, 4, 4, LDR, true>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
            else
                leaf_cat_chunk<NC, 4, 4, 4, LDR, true>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        } else if (ic <= 16)
            leaf_cat_chunk<NC, 1, 4, NW, LDR, CPX>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        else if (ic <= 32)
            leaf_cat_chunk<NC, 2, 4, NW, LDR, CPX>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        else if (NW == 4 && NC % 2 == 0 && ic <= 48 && mc > 8 * NC) {
            // two waves per column half: equal work for three row tiles
            constexpr int HC = NC > 1 ? NC / 2 : 1;
            const int ch = 16 * HC * (w >> 1);
            leaf_cat_chunk<HC, 3, 2, 2, LDR, CPX>(a, w & 1, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0 + ch, xc - ch, xrow,
                                                  red + ch);
        }
        else if (NW == 4)  // two waves per 32 rows
            leaf_cat_chunk<NC, 2, 2, 2, LDR, CPX>(a, w & 1, lr, lq, t, nb, vb, rn, nt2, i0 + 32 * (w >> 1),
                                                  w < 2 ? 32 : ic - 32, j0, xc, xrow, red + (w >> 1) * 32 * LDR);
        else if constexpr (NW == 2) {
            if (ic <= 48)
                leaf_cat_chunk<NC, 3, 2, 2, LDR, CPX>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
            else
                leaf_cat_chunk<NC, 4, 2, 2, LDR, CPX>(a, w, lr, lq, t, nb, vb, rn, nt2, i0, ic, j0, xc, xrow, red);
        }
        for (int x = tid; x < ic * MC; x += 64 * NW) {
            const int i = x / MC, j = x - i * MC;
            if (j < mc) {
                int64_t row = r0 + i0 + i;
                if (!a.tree_order) row = a.perm[row];
                double *y = &a.Y[row * a.ldy + j0 + j];
                const double v = a.alpha * red[i * LDR + j];
                *y = (a.beta == 0.0) ? v : a.beta * *y + v;
            }
        }
        __syncthreads();
    }
}

// one (leaf, column slab) slot: slot & 7 is the XCD, whose leaves form one contiguous
// eighth (taken in the order of a.order: the most work first); the slabs of one leaf are
// consecutive slots of one XCD, so its near blocks come from HBM once.
template <int NC, int NW, bool CPX>
__device__ inline void leaf_cat_slot(int64_t slot, const LeafCatArgs &a, double *red) {
    const int32_t per_xcd = (a.L + 7) / 8;
    const int nslab = (int)((a.m + 16 * NC - 1) / (16 * NC));
    const int64_t qx = slot >> 3;
    const int32_t pos = (int32_t)((slot & 7) * per_xcd + qx / nslab);
    if (pos >= a.L) return;
    const int32_t l = a.order[pos];
    const int64_t j0 = (qx % nslab) * (16 * NC);
    int tid = threadIdx.x;
    // 64 columns: the thread's number is opaque in each slot, as the offsets of every form would else be
    // computed before the loop over slots and held across it (20 registers spilled)
    if (NC == 4) asm volatile("" : "+v"(tid));
    if (NC == 4 && a.m - j0 <= 32)
        leaf_cat_slab<2, NW, CPX>(l, j0, a, red, tid);
    else if (NC == 4 && a.m - j0 <= 48)
        leaf_cat_slab<3, NW, CPX>(l, j0, a, red, tid);
    else
        leaf_cat_slab<NC, NW, CPX>(l, j0, a, red, tid);
}

// ---- the near-field term of d ell ----
//
// sum over leaves t of <dY|_t, sum_{(t,s) near} G_ts X|_s> with G_ts[i][c] =
// dg/dell(x_i, x_c) = (r / ell^2) exp(-r / ell) = (r / ell^2) N_ts[i][c] for the exponential
// kernel (the shift on the diagonal sits where r = 0): the near-field contraction of the leaf
// stage with the stored N scaled by r / ell^2 (r from the points, tree order).  Same slots,
// near-row table, row groups and rounds as leaf_cat_slot; returns the work-group's partial
// sum of the dot product (the same value in every thread).
struct DellArgs {
    const double *pts;  // n x 3, tree order
    double inv_ell, inv_ell2;
    const double *dYt;  // n x ldt, tree order
    int64_t ldt;
};

template <int NP>
struct DellRound {
    dbl2c a[NP][4];
    double c[4][3];  // coordinates of the near row's point of each k-step
    double n[2][4];  // the stored near-field entries (row tile of the wave, k-step)
    int ok[4];
};

template <int NP>
__device__ inline double leaf_dell_slot(int64_t slot, const LeafCatArgs &a, const DellArgs &d, double *red,
                                        int32_t *xrow) {
    constexpr int MC = 32 * NP, LDR = MC + 1;
    __shared__ double part_red[256];
    const int32_t per_xcd = (a.L + 7) / 8;
    const int nslab = (int)((a.m + MC - 1) / MC);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 15,
              lq = lane >> 4;
    const int64_t qx = slot >> 3;
    const int32_t pos = (int32_t)((slot & 7) * per_xcd + qx / nslab);
    if (pos >= a.L) return 0.0;
    const int32_t l = a.order[pos];
    const int32_t t = a.leaves[l];
    const int nt = a.size[t];
    const int64_t nt2 = pad_rows(nt), r0 = a.first[t];
    const int64_t j0 = (qx % nslab) * MC;
    const int mc = (int)min<int64_t>(MC, a.m - j0);
    const int64_t q0 = a.near_ptr[l];
    const int nnear = (int)(a.near_ptr[l + 1] - q0);
    const int32_t rn =
        nnear > 0 ? cat_build_rows(xrow, q0, nnear, nt2, a.near_col, a.near_off, a.first, a.size, threadIdx.x) : 0;
    const int RT = (rn + 15) >> 4;
    const double *nb = nnear > 0 ? a.Nt + a.near_off[q0] : a.Nt;
    const int xc = (mc - 1) & ~1;
    double mine = 0.0;

    for (int i0 = 0; i0 < nt; i0 += 64) {
        const int ic = min(64, nt - i0);
        const int ntile = (ic + 15) >> 4;
        const int G = ntile > 2 ? 2 : 4;
        const int wr = w / G, g = w - wr * G;
        const int tl0 = 2 * wr;
        const bool t0 = tl0 < ntile, t1 = tl0 + 1 < ntile;
        const int64_t pa = r0 + i0 + min(16 * tl0 + lr, ic - 1), pb = r0 + i0 + min(16 * tl0 + 16 + lr, ic - 1);
        const double ax = d.pts[3 * pa], ay = d.pts[3 * pa + 1], az = d.pts[3 * pa + 2];
        const double bx = d.pts[3 * pb], by = d.pts[3 * pb + 1], bz = d.pts[3 * pb + 2];

        dbl4c acc[2 * NP][2];
#pragma unroll
        for (int J = 0; J < 2 * NP; ++J) acc[J][0] = acc[J][1] = dbl4c{0.0, 0.0, 0.0, 0.0};

        auto load = [&](int r, DellRound<NP> &R) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 16 * r + 4 * u + lq, cc = min(c, rn - 1);
                R.ok[u] = c < rn;
                const int64_t xr = xrow[cc];
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    R.a[p][u] = *(const dbl2c *)(a.Xt + j0 + xr * a.ldxt + min(32 * p + 2 * lr, xc));
#pragma unroll
                for (int q = 0; q < 3; ++q) R.c[u][q] = d.pts[3 * xr + q];
                R.n[0][u] = nb[(int64_t)cc * nt2 + (pa - r0)];
                R.n[1][u] = nb[(int64_t)cc * nt2 + (pb - r0)];
            }
        };
        auto gval = [&](double x, double y, double z, const double *c, double nv) {
            const double dx = x - c[0], dy = y - c[1], dz = z - c[2];
            const double r = sqrt(dx * dx + dy * dy + dz * dz);
            return (r * d.inv_ell2) * nv;
        };
        auto multiply = [&](DellRound<NP> &R) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double g0 = t0 ? gval(ax, ay, az, R.c[u], R.n[0][u]) : 0.0;
                const double g1 = t1 ? gval(bx, by, bz, R.c[u], R.n[1][u]) : 0.0;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const dbl2c v = R.ok[u] ? R.a[p][u] : dbl2c{0.0, 0.0};
#pragma unroll
                    for (int hj = 0; hj < 2; ++hj) {
                        if (t0)
                            acc[2 * p + hj][0] =
                                __builtin_amdgcn_mfma_f64_16x16x4f64(v[hj], g0, acc[2 * p + hj][0], 0, 0, 0);
                        if (t1)
                            acc[2 * p + hj][1] =
                                __builtin_amdgcn_mfma_f64_16x16x4f64(v[hj], g1, acc[2 * p + hj][1], 0, 0, 0);
                    }
                }
            }
        };
        if (g < RT) {
            const int last = g + ((RT - 1 - g) / G) * G;
            DellRound<NP> s0, s1, s2;
            int r = g;
            load(r, s0);
            load(min(r + G, last), s1);
            for (;;) {
                load(min(r + 2 * G, last), s2);
                multiply(s0);
                r += G;
                if (r > last) break;
                load(min(r + 2 * G, last), s0);
                multiply(s1);
                r += G;
                if (r > last) break;
                load(min(r + 2 * G, last), s1);
                multiply(s2);
                r += G;
                if (r > last) break;
            }
        }
        for (int gg = 0; gg < G; ++gg) {
            if (g == gg)
#pragma unroll
                for (int J = 0; J < 2 * NP; ++J)
#pragma unroll
                    for (int I = 0; I < 2; ++I)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int col = 32 * (J >> 1) + 2 * (lq + 4 * q) + (J & 1);
                            const int row = 16 * (tl0 + I) + lr;
                            double *cell = &red[row * LDR + col];
                            *cell = (gg == 0) ? acc[J][I][q] : *cell + acc[J][I][q];
                        }
            __syncthreads();
        }
        // <dY|_t, G X> over the chunk's rows and the slab's columns
        for (int x = threadIdx.x; x < ic * MC; x += 256) {
            const int i = x / MC, j = x - i * MC;
            if (j < mc) mine += red[i * LDR + j] * d.dYt[(r0 + i0 + i) * d.ldt + j0 + j];
        }
        __syncthreads();
    }
    // the work-group's sum in a fixed order
    part_red[threadIdx.x] = mine;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part_red[threadIdx.x] += part_red[threadIdx.x + h];
        __syncthreads();
    }
    const double tot = part_red[0];
    __syncthreads();
    return tot;
}

// near-field term of d ell: one slot per work-group, part[blockIdx.x] = its partial sum
template <int NP>
__global__ __launch_bounds__(256, 2) void k_dell_near(LeafCatArgs a, DellArgs d, double *__restrict__ part) {
    __shared__ double red[64 * (32 * NP + 1)];
    extern __shared__ int32_t xrow[];
    const double tot = leaf_dell_slot<NP>(blockIdx.x, a, d, red, xrow);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// the leaf stage over slots [slot0, slot1): dynamic LDS = the near-row table and the partial tiles
template <int NC, int NW, bool CPX>
__global__ __launch_bounds__(64 * NW, (NC == 1 || (NW == 4 && NC == 2)) && !CPX ? 3 : 2) void k_leaf_cat(LeafCatArgs a, int64_t slot0, int64_t slot1) {
    extern __shared__ double red[];
    for (int64_t slot = slot0 + blockIdx.x; slot < slot1; slot += gridDim.x) leaf_cat_slot<NC, NW, CPX>(slot, a, red);
}

// calls f(k_leaf_cat<..>) for the column tiles, waves and kind of operator of one launch
// (two waves: nc = 2, real operators; complex operators: nc <= 2)
template <typename F>
void leaf_cat_kernel(int nc, bool two, bool cplx, F f) {
    if (cplx) return nc == 1 ? f(&k_leaf_cat<1, 4, true>, 256) : f(&k_leaf_cat<2, 4, true>, 256);
    if (two) return f(&k_leaf_cat<2, 2, false>, 128);
    switch (nc) {
        case 1: return f(&k_leaf_cat<1, 4, false>, 256);
        case 2: return f(&k_leaf_cat<2, 4, false>, 256);
        case 3: return f(&k_leaf_cat<3, 4, false>, 256);
        default: return f(&k_leaf_cat<4, 4, false>, 256);
    }
}

// A transfer level with a share of the near field beside it: work-groups [0, items) run the
// level (item i: list entry i / gy, column slab i % gy), work-group items + lead + s runs
// leaf slot slot0 + s with near = 1, basis = 0 (the near field needs only X); the `lead`
// idle work-groups put slot s on XCD s % 8 (work-groups are dealt to the XCDs in turn), as
// in the leaf stage's own launch.  The level's chain of dependent launches then overlaps
// streaming near-field work.  Dynamic LDS: the larger of the level's operand tiles and the
// leaf work's buffers.
template <int NJ, int NP, int UP>
__global__ __launch_bounds__(256, 2) void k_level_near(int64_t items, int gy, int64_t m, const int32_t *__restrict__ list,
                                                       const int32_t *__restrict__ aux, const double *__restrict__ E,
                                                       double *__restrict__ hat, int64_t ldh, Skip skip,
                                                       LeafCatArgs a, int64_t slot0, int lead) {
    extern __shared__ double lds[];
    const int64_t b = blockIdx.x;
    if (b < items) {
        const int i = (int)(b / gy), by = (int)(b - (int64_t)i * gy);
        if (UP)
            up64_item<NJ>(i, by, m, list, aux, E, hat, ldh, skip, lds);
        else
            down64_item<NJ>(i, by, m, list, aux, E, hat, ldh, skip, lds);
    } else if (b >= items + lead) {
        leaf_cat_slot<2 * NP, 4, false>(slot0 + (b - items - lead), a, lds);
    }
}

}  // namespace mfma
}  // namespace h2x
