// Transfer passes of the FP64 operator through the tensor structure of the transfer matrices
// (Chebyshev order P = 1 to 8, rank k = P^3).  The interpolation nodes of a cluster form a
// P x P x P Chebyshev grid on its axis-parallel box and the Lagrange polynomials are products
// of one-dimensional ones, so the transfer matrix of a son c (the father's polynomials at the
// son's nodes) is the Kronecker product of three P x P matrices:
//
//   E_c[a, nu] = F_c^0[a0, nu0] F_c^1[a1, nu1] F_c^2[a2, nu2],   a = a0 + P a1 + P^2 a2,
//
// F_c^d[i, j] = the father's j-th Lagrange polynomial on axis d at the son's i-th node on that
// axis (stored as 3 P^2 doubles per cluster, [d][P i + j]).  The upward step
// x_t = sum_c E_c^T x_c and the downward step y_c += E_c y_t then take three passes of P-term
// sums over the k entries of a column (3 P^4 multiply-adds instead of P^6: 768 instead of 4096
// at P = 4) and read 3 P^2 factors instead of the k^2 entries of E_c.
//
// One work-group of 256 threads per (cluster, slab of MC columns): the input columns go to LDS
// (k rows of MC + 1 doubles per block); a pass maps each P-entry pencil along its axis to a
// thread, which overwrites it in place (pencils are disjoint: no barrier inside a pass);
// consecutive threads take consecutive columns, so LDS rows are read without bank conflicts.
// The last pass reads LDS and writes (upward) or adds to (downward) the output in HBM.
#pragma once

#include <vector>

#include "device.hpp"

namespace h2x {
namespace kron {

// rows of the P-entry pencil o (0..P^2-1: the two digits other than axis d, the lower one
// first) along axis d: base + stride * l, l = 0..P-1
template <int P>
__device__ inline int pencil_base(int d, int o) {
    return d == 0 ? P * o : (d == 1 ? (o % P) + P * P * (o / P) : o);
}
template <int P>
__device__ inline int axis_stride(int d) { return d == 0 ? 1 : (d == 1 ? P : P * P); }

// v' = M v on every pencil along axis d of NQ blocks in LDS; M = (F^d)^T (TR, upward) or F^d.
// tid: thread of the 256 that share the blocks
template <int P, int MC, int NQ, bool TR>
__device__ inline void pass(double *buf, const double *fs, int d, int tid) {
    constexpr int K = P * P * P, LD = MC + 1, NPEN = NQ * P * P * MC;
    const int st = axis_stride<P>(d);
#pragma unroll
    for (int u = 0; u < (NPEN + 255) / 256; ++u) {
        const int idx = tid + 256 * u;
        if (NPEN % 256 != 0 && idx >= NPEN) break;
        const int j = idx % MC, pen = idx / MC, q = pen / (P * P);
        double *col = buf + (q * K + pencil_base<P>(d, pen % (P * P))) * LD + j;
        const double *F = fs + q * 3 * P * P + P * P * d;
        double v[P], o[P];
#pragma unroll
        for (int l = 0; l < P; ++l) v[l] = col[st * l * LD];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < P; ++l) s += (TR ? F[P * l + i] : F[P * i + l]) * v[l];
            o[i] = s;
        }
#pragma unroll
        for (int i = 0; i < P; ++i) col[st * i * LD] = o[i];
    }
}

// ---- the steps of one cluster, shared by the level and the group kernels ----

// x_{sc[q]} -> LDS
template <int P, int MC>
__device__ inline void up_load(double *buf, const int32_t (&sc)[2], const double *xh, int64_t ldh, int64_t j0, int mc,
                               int tid) {
    constexpr int K = P * P * P, LD = MC + 1, NIN = 2 * K * MC;
#pragma unroll
    for (int u = 0; u < (NIN + 255) / 256; ++u) {
        const int idx = tid + 256 * u;
        if (NIN % 256 != 0 && idx >= NIN) break;
        const int j = idx % MC, r = (idx / MC) % K, q = idx / (MC * K);
        buf[(q * K + r) * LD + j] = xh[((int64_t)sc[q] * K + r) * ldh + j0 + min(j, mc - 1)];
    }
}

// axis 2 and the sum over the two sons
template <int P, int MC>
__device__ inline void up_store(const double *buf, const double *fs, int32_t t, double *xh, int64_t ldh, int64_t j0,
                                int mc, int tid) {
    constexpr int K = P * P * P, LD = MC + 1, NF = 3 * P * P, NOUT = P * P * MC;
#pragma unroll
    for (int u = 0; u < (NOUT + 255) / 256; ++u) {
        const int idx = tid + 256 * u;
        if (NOUT % 256 != 0 && idx >= NOUT) break;
        const int j = idx % MC, o = idx / MC;
        double acc[P];
#pragma unroll
        for (int i = 0; i < P; ++i) acc[i] = 0.0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double *F = fs + q * NF + 2 * P * P;
            double v[P];
#pragma unroll
            for (int l = 0; l < P; ++l) v[l] = buf[(q * K + o + P * P * l) * LD + j];
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
                for (int l = 0; l < P; ++l) acc[i] += F[P * l + i] * v[l];
        }
        if (j < mc)
#pragma unroll
            for (int i = 0; i < P; ++i) xh[((int64_t)t * K + o + P * P * i) * ldh + j0 + j] = acc[i];
    }
}

// y_p -> LDS
template <int P, int MC>
__device__ inline void down_load(double *buf, int32_t p, const double *yh, int64_t ldh, int64_t j0, int mc, int tid) {
    constexpr int K = P * P * P, LD = MC + 1, NIN = K * MC;
#pragma unroll
    for (int u = 0; u < (NIN + 255) / 256; ++u) {
        const int idx = tid + 256 * u;
        if (NIN % 256 != 0 && idx >= NIN) break;
        const int j = idx % MC, r = idx / MC;
        buf[r * LD + j] = yh[((int64_t)p * K + r) * ldh + j0 + min(j, mc - 1)];
    }
}

// axis 2, added to y_c
template <int P, int MC>
__device__ inline void down_store(const double *buf, const double *fs, int32_t c, double *yh, int64_t ldh, int64_t j0,
                                  int mc, int tid) {
    constexpr int K = P * P * P, LD = MC + 1, NOUT = P * P * MC;
#pragma unroll
    for (int u = 0; u < (NOUT + 255) / 256; ++u) {
        const int idx = tid + 256 * u;
        if (NOUT % 256 != 0 && idx >= NOUT) break;
        const int j = idx % MC, o = idx / MC;
        const double *F = fs + 2 * P * P;
        double v[P];
#pragma unroll
        for (int l = 0; l < P; ++l) v[l] = buf[(o + P * P * l) * LD + j];
        if (j < mc)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                double s = 0.0;
#pragma unroll
                for (int l = 0; l < P; ++l) s += F[P * i + l] * v[l];
                yh[((int64_t)c * K + o + P * P * i) * ldh + j0 + j] += s;
            }
    }
}

// x_t = E_{s0}^T x_{s0} + E_{s1}^T x_{s1} for the clusters list[i] with sons son[2 i], son[2 i + 1]
template <int P, int MC>
__global__ __launch_bounds__(256) void k_up(int64_t m, const int32_t *__restrict__ list,
                                            const int32_t *__restrict__ son, const double *__restrict__ F1,
                                            double *__restrict__ xh, int64_t ldh, Skip skip) {
    constexpr int K = P * P * P, LD = MC + 1, NF = 3 * P * P;
    __shared__ double buf[2 * K * LD];
    __shared__ double fs[2 * NF];
    const int32_t t = list[blockIdx.x];
    if (skip(t)) return;
    const int32_t sc[2] = {son[2 * blockIdx.x], son[2 * blockIdx.x + 1]};
    const int64_t j0 = (int64_t)blockIdx.y * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    for (int e = threadIdx.x; e < 2 * NF; e += 256) fs[e] = F1[(int64_t)sc[e / NF] * NF + e % NF];
    up_load<P, MC>(buf, sc, xh, ldh, j0, mc, threadIdx.x);
    __syncthreads();
    pass<P, MC, 2, true>(buf, fs, 0, threadIdx.x);
    __syncthreads();
    pass<P, MC, 2, true>(buf, fs, 1, threadIdx.x);
    __syncthreads();
    up_store<P, MC>(buf, fs, t, xh, ldh, j0, mc, threadIdx.x);
}

// y_c += E_c y_{par} for the clusters list[i] with fathers par[i]
template <int P, int MC>
__global__ __launch_bounds__(256) void k_down(int64_t m, const int32_t *__restrict__ list,
                                              const int32_t *__restrict__ par, const double *__restrict__ F1,
                                              double *__restrict__ yh, int64_t ldh, Skip skip) {
    constexpr int K = P * P * P, LD = MC + 1, NF = 3 * P * P;
    __shared__ double buf[K * LD];
    __shared__ double fs[NF];
    const int32_t c = list[blockIdx.x], p = par[blockIdx.x];
    if (skip(c)) return;
    const int64_t j0 = (int64_t)blockIdx.y * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    for (int e = threadIdx.x; e < NF; e += 256) fs[e] = F1[(int64_t)c * NF + e];
    down_load<P, MC>(buf, p, yh, ldh, j0, mc, threadIdx.x);
    __syncthreads();
    pass<P, MC, 1, false>(buf, fs, 0, threadIdx.x);
    __syncthreads();
    pass<P, MC, 1, false>(buf, fs, 1, threadIdx.x);
    __syncthreads();
    down_store<P, MC>(buf, fs, c, yh, ldh, j0, mc, threadIdx.x);
}

// ---- up to three small levels in one launch ----
//
// A level of few work-groups costs its launch and a chain of cold loads (about 4.5 us) for half
// a microsecond of work.  Here a work-group of four groups of 256 threads takes the subtree of one
// cluster over nlev levels: 4, 2 and 1 clusters (upward; downward 1, 2 and 4), one per group, all
// list entries and factors loaded at the start, the hats handed on through the CU's cache.
// rng[4 e ..]: for entry e of the level lists, the ranges of entries of its subtree one level
// deeper and two levels deeper.  The same sums as the level kernels.
// Chosen by kUpGroupItems and kDownGroupItems (measurements there).

template <int P>
__global__ __launch_bounds__(1024) void k_up_group(int64_t m, int32_t e0, int nlev, const int32_t *__restrict__ list,
                                                   const int32_t *__restrict__ son, const int32_t *__restrict__ rng,
                                                   const double *__restrict__ F1, double *xh, int64_t ldh, Skip skip) {
    constexpr int MC = 16, K = P * P * P, LD = MC + 1, NF = 3 * P * P;
    __shared__ double bufs[4][2 * K * LD];
    __shared__ double fss[4][3][2 * NF];
    const int32_t e = e0 + blockIdx.x;
    if (skip(list[e])) return;
    const int tid = threadIdx.x & 255, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int64_t j0 = (int64_t)blockIdx.y * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    int32_t t[3], sc[3][2];
#pragma unroll
    for (int l = 0; l < 3; ++l) {  // group g's entry l levels below the root
        const int32_t a = l == 0 ? e : rng[4 * e + 2 * (l - 1)], b = l == 0 ? e + 1 : rng[4 * e + 2 * (l - 1) + 1];
        const bool in = l < nlev && a + g < b;
        const int32_t i = in ? a + g : e;
        t[l] = in ? list[i] : -1;
        sc[l][0] = son[2 * i];
        sc[l][1] = son[2 * i + 1];
    }
    double *buf = bufs[g];
#pragma unroll
    for (int l = 0; l < 3; ++l)
        if (t[l] >= 0)
            for (int x = tid; x < 2 * NF; x += 256) fss[g][l][x] = F1[(int64_t)sc[l][x / NF] * NF + x % NF];
#pragma unroll
    for (int l = 2; l >= 0; --l) {
        if (l >= nlev) continue;
        const bool in = t[l] >= 0;
        if (in) up_load<P, MC>(buf, sc[l], xh, ldh, j0, mc, tid);
        __syncthreads();
        if (in) pass<P, MC, 2, true>(buf, fss[g][l], 0, tid);
        __syncthreads();
        if (in) pass<P, MC, 2, true>(buf, fss[g][l], 1, tid);
        __syncthreads();
        if (in) up_store<P, MC>(buf, fss[g][l], t[l], xh, ldh, j0, mc, tid);
        __syncthreads();
    }
}

template <int P>
__global__ __launch_bounds__(1024) void k_down_group(int64_t m, int32_t e0, int nlev, const int32_t *__restrict__ list,
                                                     const int32_t *__restrict__ par, const int32_t *__restrict__ rng,
                                                     const double *__restrict__ F1, double *yh, int64_t ldh, Skip skip) {
    constexpr int MC = 16, K = P * P * P, LD = MC + 1, NF = 3 * P * P;
    __shared__ double bufs[4][K * LD];
    __shared__ double fss[4][3][NF];
    const int32_t e = e0 + blockIdx.x;
    if (skip(list[e])) return;
    const int tid = threadIdx.x & 255, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int64_t j0 = (int64_t)blockIdx.y * MC;
    const int mc = (int)min<int64_t>(MC, m - j0);
    int32_t c[3], pr[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const int32_t a = l == 0 ? e : rng[4 * e + 2 * (l - 1)], b = l == 0 ? e + 1 : rng[4 * e + 2 * (l - 1) + 1];
        const bool in = l < nlev && a + g < b;
        const int32_t i = in ? a + g : e;
        c[l] = in ? list[i] : -1;
        pr[l] = par[i];
    }
    double *buf = bufs[g];
#pragma unroll
    for (int l = 0; l < 3; ++l)
        if (c[l] >= 0)
            for (int x = tid; x < NF; x += 256) fss[g][l][x] = F1[(int64_t)c[l] * NF + x];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        if (l >= nlev) break;
        const bool in = c[l] >= 0;
        if (in) down_load<P, MC>(buf, pr[l], yh, ldh, j0, mc, tid);
        __syncthreads();
        if (in) pass<P, MC, 1, false>(buf, fss[g][l], 0, tid);
        __syncthreads();
        if (in) pass<P, MC, 1, false>(buf, fss[g][l], 1, tid);
        __syncthreads();
        if (in) down_store<P, MC>(buf, fss[g][l], c[l], yh, ldh, j0, mc, tid);
        __syncthreads();
    }
}

// ---- launches: all upward levels dhi .. dlo, all downward levels dlo .. dhi ----

// levels of at most this many (cluster, 16-column slab) items go in groups of up to three (upward /
// downward pass in us, level by level -> grouped): k = 27, n = 4096, 4 columns 18.7 / 17.9 ->
// 13.6 / 15.0; 32 columns of a cube of 16000 26.6 / 28.3 -> 17.6 / 24.7; k = 64, n = 65536, 32
// columns 43.9 / 49.2 -> 42.7 / 44.1.  A step of the upward kernel at k = 64 is long enough that
// larger levels lose (512 items: matvec 36.5 -> 38.5), at k = 125 every level does (34 -> 39.6).
template <int P>
constexpr int64_t kUpGroupItems = P <= 3 ? 1024 : (P == 4 ? 256 : 0);
template <int P>
constexpr int64_t kDownGroupItems = P <= 3 ? 1024 : (P <= 5 ? 2048 : 0);
// wider levels with fewer work-groups than this (clusters x column slabs) take 16-column slabs:
// more work-groups with half the work each shorten a level that is one wave of work-groups
constexpr int64_t kNarrowLevel = 256;

// MC: columns per work-group of a level of its own
template <int P, int MC>
void up_levels(const DevMat &dm, int64_t m, int dhi, int dlo, double *xh, int64_t ldh, hipStream_t st, Skip skip) {
    const std::vector<int32_t> &ptr = dm.plan->lvl_inner_ptr;
    const int64_t s16 = (m + 15) / 16, smc = (m + MC - 1) / MC;
    for (int d = dhi; d >= dlo;) {
        const int32_t b = ptr[d], e = ptr[d + 1];
        if constexpr (kUpGroupItems<P> > 0) {
            int nlev = 0;  // levels d, d - 1, d - 2 that are small
            while (nlev < 3 && d - nlev >= dlo && (ptr[d - nlev + 1] - ptr[d - nlev]) * s16 <= kUpGroupItems<P>) ++nlev;
            if (nlev > 1) {
                const int root = d - nlev + 1;
                const int32_t n0 = ptr[root + 1] - ptr[root];
                if (n0 > 0)
                    hipLaunchKernelGGL((k_up_group<P>), dim3((unsigned)n0, (unsigned)s16), dim3(1024), 0, st, m,
                                       ptr[root], nlev, dm.lvl_inner, dm.up_son, dm.up_rng, dm.E1, xh, ldh, skip);
                d = root - 1;
                continue;
            }
        }
        if (e > b && MC > 16 && (e - b) * smc < kNarrowLevel)
            hipLaunchKernelGGL((k_up<P, 16>), dim3(e - b, (unsigned)s16), dim3(256), 0, st, m, dm.lvl_inner + b,
                               dm.up_son + 2 * b, dm.E1, xh, ldh, skip);
        else if (e > b)
            hipLaunchKernelGGL((k_up<P, MC>), dim3(e - b, (unsigned)smc), dim3(256), 0, st, m, dm.lvl_inner + b,
                               dm.up_son + 2 * b, dm.E1, xh, ldh, skip);
        --d;
    }
}

template <int P, int MC>
void down_levels(const DevMat &dm, int64_t m, int dlo, int dhi, double *yh, int64_t ldh, hipStream_t st, Skip skip) {
    const std::vector<int32_t> &ptr = dm.plan->lvl_ptr;
    const int64_t s16 = (m + 15) / 16, smc = (m + MC - 1) / MC;
    for (int d = dlo; d <= dhi;) {
        const int32_t b = ptr[d], e = ptr[d + 1];
        if constexpr (kDownGroupItems<P> > 0) {
            int nlev = 0;  // levels d, d + 1, d + 2 that are small
            while (nlev < 3 && d + nlev <= dhi && (ptr[d + nlev + 1] - ptr[d + nlev]) * s16 <= kDownGroupItems<P>)
                ++nlev;
            if (nlev > 1) {
                if (e > b)
                    hipLaunchKernelGGL((k_down_group<P>), dim3(e - b, (unsigned)s16), dim3(1024), 0, st, m, b, nlev,
                                       dm.lvl_all, dm.dn_par, dm.dn_rng, dm.E1, yh, ldh, skip);
                d += nlev;
                continue;
            }
        }
        if (e > b && MC > 16 && (e - b) * smc < kNarrowLevel)
            hipLaunchKernelGGL((k_down<P, 16>), dim3(e - b, (unsigned)s16), dim3(256), 0, st, m, dm.lvl_all + b,
                               dm.dn_par + b, dm.E1, yh, ldh, skip);
        else if (e > b)
            hipLaunchKernelGGL((k_down<P, MC>), dim3(e - b, (unsigned)smc), dim3(256), 0, st, m, dm.lvl_all + b,
                               dm.dn_par + b, dm.E1, yh, ldh, skip);
        ++d;
    }
}

// MC16: columns per work-group in 16s (1 to 4; orders above 4 hold 16 columns)
template <int MC16>
void up_levels_p(const DevMat &dm, int64_t m, int dhi, int dlo, double *xh, int64_t ldh, hipStream_t st, Skip skip) {
    switch (dm.p) {
        case 1: up_levels<1, 16 * MC16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 2: up_levels<2, 16 * MC16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 3: up_levels<3, 16 * MC16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 4: up_levels<4, 16 * MC16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 5: up_levels<5, 16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 6: up_levels<6, 16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        case 7: up_levels<7, 16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
        default: up_levels<8, 16>(dm, m, dhi, dlo, xh, ldh, st, skip); break;
    }
}
template <int MC16>
void down_levels_p(const DevMat &dm, int64_t m, int dlo, int dhi, double *yh, int64_t ldh, hipStream_t st, Skip skip) {
    switch (dm.p) {
        case 1: down_levels<1, 16 * MC16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 2: down_levels<2, 16 * MC16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 3: down_levels<3, 16 * MC16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 4: down_levels<4, 16 * MC16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 5: down_levels<5, 16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 6: down_levels<6, 16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        case 7: down_levels<7, 16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
        default: down_levels<8, 16>(dm, m, dlo, dhi, yh, ldh, st, skip); break;
    }
}

}  // namespace kron
}  // namespace h2x
