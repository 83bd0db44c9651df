// Coupling stage of the FP64 operator for the ranks k = P^3 <= 27 (P = 1, 2, 3):
//   y_t = sum_{(t,s) in C_t, admissible} S_b x_s     for every row cluster t.
//
// One wave works alone on a row cluster and a slab of 16 NJ columns: it loads NB consecutive
// blocks of its list (row-major S_b, contiguous over the list) and their x_s into registers with
// whole-line loads, one step ahead, puts them into its own stretch of LDS, and multiplies from
// there with v_mfma_f64_16x16x4f64.  LDS operations of a wave complete in the order in which they
// are issued and wave_sync keeps the compiler from changing it, so a step needs neither a
// work-group barrier nor a second buffer.  The list's steps are cut into four consecutive parts
// whose sums are added in order, either by the four waves of a work-group, a part each (SP = 4: a
// quarter of the serial chain), or by one wave, part after part (SP = 1: four units to a
// work-group).  So every launch shape gives the same bits, and a system solved in a batch those
// of the system alone.
//
// Bound by the loads of S_b and x_s (a 27 x 27 block has 5.8 KB, its x_s 3.5 KB at 16 columns).
// Reading S_b straight into operand registers (8 bytes per lane, rows 216 bytes apart, every line
// touched by several instructions) and sharing x_s over two waves behind a barrier was slower
// throughout: k = 27, 16 columns, sphere, n = 4096 60 -> 21 us, n = 32000 192 -> 96 us; cube,
// n = 32000, 32 columns 556 -> 280 us; k = 8, n = 16000 84 -> 18 us.
#pragma once

#include <algorithm>
#include <type_traits>

#include "device.hpp"

namespace h2x {

typedef double dbl4 __attribute__((ext_vector_type(4)));

template <int P, int NJ, int SP>
__global__ __launch_bounds__(256) void k_coupling_small(
    int64_t m, int32_t C, int32_t rows_per_xcd, const int32_t *__restrict__ order, const int64_t *__restrict__ adm_ptr,
    const int32_t *__restrict__ adm_col, const double *__restrict__ S, const double *__restrict__ xh,
    double *__restrict__ yh, int64_t ldh, Skip skip, int jpass) {
    constexpr int K = P * P * P, NT = (K + 15) / 16, KS = (K + 3) / 4;  // row tiles, k-steps of a block
    constexpr int NB = P == 3 ? 1 : 4;                                  // blocks per step
    constexpr int MC = 16 * NJ, W = 4;
    constexpr int SN = NB * K * K, SU = (SN + 63) / 64;                 // S entries of a step, loads per lane
    constexpr int XN = NB * 4 * KS * MC, XU = (XN + 63) / 64;           // x entries (rows past K zero)
    constexpr int SL = SU * 64, WL = SL + XU * 64;                      // LDS doubles per wave
    constexpr int RL = SP > 1 ? NT * NJ * 256 : 0;                      // partial sums of a wave
    __shared__ double lds[W * (WL > RL ? WL : RL)];
    const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nslab = (int)((m + MC - 1) / MC);
    const int unit = SP == 1 ? (int)(blockIdx.x >> 3) * 4 + w : (int)(blockIdx.x >> 3);
    const int pos = unit / nslab, slot = (blockIdx.x & 7) * rows_per_xcd + pos;
    // (no barrier when SP = 1; with SP > 1 the whole work-group has the same unit)
    if (pos >= rows_per_xcd || slot >= C) return;
    const int32_t t = order[slot];
    if (skip(t)) return;
    const int64_t j0 = (int64_t)(unit % nslab) * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    const int64_t b0 = adm_ptr[t];
    const int nb = (int)(adm_ptr[t + 1] - b0), steps = (nb + NB - 1) / NB;
    const int quarter = (steps + 3) / 4;
    const int first = SP == 1 ? 0 : min(steps, w * quarter), last = SP == 1 ? steps : min(steps, (w + 1) * quarter);
    double *ss = lds + w * WL, *xs = ss + SL;

    dbl4 acc[NT][NJ];
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
        for (int J = 0; J < NJ; ++J) acc[I][J] = dbl4{0.0, 0.0, 0.0, 0.0};

    if (first < last) {
        double sv[SU], xv[XU];
        // every load unconditional from a clamped address: entries past the list re-read its last
        // one and meet zero rows of x
        auto load = [&](int i) {
            const int left = nb - i * NB;  // blocks from this step to the end of the list
            const double *Sb = S + (b0 + (int64_t)i * NB) * (K * K);
            const int lim = min(NB, left) * K * K - 1;
#pragma unroll
            for (int u = 0; u < SU; ++u) sv[u] = __builtin_nontemporal_load(Sb + min(lane + 64 * u, lim));
            const double *src[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)
                src[q] = xh + (int64_t)adm_col[b0 + min(i * NB + q, nb - 1)] * K * ldh + j0;
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int e = lane + 64 * u, c = e % MC, row = e / MC, q = row / (4 * KS), r = row % (4 * KS);
                const double *p = src[0];
#pragma unroll
                for (int z = 1; z < NB; ++z) p = q >= z ? src[z] : p;
                // jpass: column c takes its partner c ^ 1 (J x = (-im, re) per complex column)
                xv[u] = p[(int64_t)min(r, K - 1) * ldh + ((c < mc ? c : 0) ^ jpass)];
            }
        };
        auto store = [&](int i) {
            const int left = nb - i * NB;
#pragma unroll
            for (int u = 0; u < SU; ++u) ss[lane + 64 * u] = sv[u];
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int e = lane + 64 * u, c = e % MC, row = e / MC, q = row / (4 * KS), r = row % (4 * KS);
                const double v = (jpass & ~c & 1) ? -xv[u] : xv[u];
                xs[e] = (r < K && c < mc && q < left) ? v : 0.0;
            }
        };
        auto multiply = [&]() {
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    double a[NT], b[NJ];
#pragma unroll
                    for (int I = 0; I < NT; ++I)
                        a[I] = ss[q * K * K + min(16 * I + lr, K - 1) * K + min(4 * kk + lq, K - 1)];
#pragma unroll
                    for (int J = 0; J < NJ; ++J) b[J] = xs[((q * KS + kk) * 4 + lq) * MC + 16 * J + lr];
#pragma unroll
                    for (int I = 0; I < NT; ++I)
#pragma unroll
                        for (int J = 0; J < NJ; ++J)
                            acc[I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[I], b[J], acc[I][J], 0, 0, 0);
                }
        };
        dbl4 sum[NT][NJ];
#pragma unroll
        for (int I = 0; I < NT; ++I)
#pragma unroll
            for (int J = 0; J < NJ; ++J) sum[I][J] = dbl4{0.0, 0.0, 0.0, 0.0};
        load(first);
        int i = first;
        for (int end = first + quarter;; end += quarter) {  // (SP = 4: one part)
            for (const int stop = min(end, last - 1); i < stop; ++i) {
                store(i);
                wave_sync();
                load(i + 1);
                multiply();
                wave_sync();
            }
            if (SP > 1 || end >= last) break;
#pragma unroll
            for (int I = 0; I < NT; ++I)
#pragma unroll
                for (int J = 0; J < NJ; ++J) {
                    sum[I][J] += acc[I][J];
                    acc[I][J] = dbl4{0.0, 0.0, 0.0, 0.0};
                }
        }
        store(i);
        wave_sync();
        multiply();
        if constexpr (SP == 1)
#pragma unroll
            for (int I = 0; I < NT; ++I)
#pragma unroll
                for (int J = 0; J < NJ; ++J) acc[I][J] = sum[I][J] + acc[I][J];
    }
    // D layout of the 16x16x4 f64 MFMA: lane l, register r -> row l / 16 + 4 r, column l % 16
    if constexpr (SP > 1) {
        __syncthreads();
        if (w > 0)
#pragma unroll
            for (int I = 0; I < NT; ++I)
#pragma unroll
                for (int J = 0; J < NJ; ++J)
#pragma unroll
                    for (int r = 0; r < 4; ++r) lds[w * RL + ((I * NJ + J) * 4 + r) * 64 + lane] = acc[I][J][r];
        __syncthreads();
        if (w > 0) return;
#pragma unroll
        for (int g = 1; g < 4; ++g)  // (an empty part adds zeros)
#pragma unroll
            for (int I = 0; I < NT; ++I)
#pragma unroll
                for (int J = 0; J < NJ; ++J)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[I][J][r] += lds[g * RL + ((I * NJ + J) * 4 + r) * 64 + lane];
    }
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
        for (int J = 0; J < NJ; ++J) {
            const int col = 16 * J + lr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * I + lq + 4 * r;
                if (col < mc && row < K) {
                    double *y = &yh[((int64_t)t * K + row) * ldh + j0 + col];
                    *y = jpass ? *y + acc[I][J][r] : acc[I][J][r];
                }
            }
        }
}

// nrows clusters in the order of rows.  One or two column tiles per work-group (more spill the
// registers that hold the loads ahead): one where 16-column units are few enough to want all of
// them (k = 27, 391 rows, 64 columns: 39 against 43 us; 1487 rows: 156 against 135 us).
// k = 27: always the four-wave form (131072 points on a sphere, 32 columns: 500 us, one wave 510;
// n = 4096: 28 against 46 us); k <= 8, whose lists are a few steps: one wave per unit once the
// units fill the chip (n = 131072, 32 columns: 158 against 181 us; n = 4096: 18 against 11 us).
inline void launch_coupling_small(const DevMat &dm, int64_t m, const double *S, const double *xh, double *yh,
                                  int64_t ldh, hipStream_t st, Skip skip, int nj_force, int32_t nrows,
                                  const int32_t *rows, int jpass) {
    if (nrows <= 0) return;
    const int32_t rpx = (nrows + 7) / 8;
    const int64_t tiles = (m + 15) / 16, units1 = nrows * tiles;
    const int nj = nj_force ? std::min(nj_force, 2) : (tiles == 1 || units1 < (dm.p == 3 ? 1600 : 12000) ? 1 : 2);
    const int64_t units = rpx * ((m + 16 * nj - 1) / (16 * nj));
    auto go = [&](auto Pc, auto NJc, auto SPc) {
        constexpr int P = decltype(Pc)::value, NJ = decltype(NJc)::value, SP = decltype(SPc)::value;
        hipLaunchKernelGGL((k_coupling_small<P, NJ, SP>), dim3((unsigned)(8 * (SP == 1 ? (units + 3) / 4 : units))),
                           dim3(256), 0, st, m, nrows, rpx, rows, dm.adm_ptr, dm.adm_col, S, xh, yh, ldh, skip, jpass);
    };
    auto with_nj = [&](auto Pc, auto SPc) {
        nj == 1 ? go(Pc, std::integral_constant<int, 1>{}, SPc) : go(Pc, std::integral_constant<int, 2>{}, SPc);
    };
    auto with_sp = [&](auto Pc) {
        units1 < 6000 ? with_nj(Pc, std::integral_constant<int, 4>{}) : with_nj(Pc, std::integral_constant<int, 1>{});
    };
    switch (dm.p) {
        case 1: with_sp(std::integral_constant<int, 1>{}); break;
        case 2: with_sp(std::integral_constant<int, 2>{}); break;
        default: with_nj(std::integral_constant<int, 3>{}, std::integral_constant<int, 4>{}); break;
    }
}

}  // namespace h2x
