// Device-side construction of the H^2 representation (section 2): Chebyshev
// tensor nodes per cluster, leaf matrices V_t, transfer matrices E_t, coupling
// matrices S_b of the admissible leaves and dense near-field blocks.  The
// operator can be tens of GB (coupling matrices dominate), so it is generated
// where it is used, directly into the caller's workspace.
#include <cmath>
#include <type_traits>

#include "device.hpp"
#include "types.hpp"

namespace h2x {

namespace {

template <typename T>
T *carve(size_t &off, char *base, size_t count) {
    off = align_up(off);
    T *ptr = base ? (T *)(base + off) : nullptr;
    off += count * sizeof(T);
    return ptr;
}

__device__ inline double kernel_g(int kernel, double ell, const double *a, const double *b) {
    if (kernel == H2X_KERNEL_EXP) {
        double dx = a[0] - b[0], dy = a[1] - b[1], dz = a[2] - b[2];
        return exp(-sqrt(dx * dx + dy * dy + dz * dz) / ell);
    }
    if (kernel == H2X_KERNEL_POLY) {
        double d = 1.0 + a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
        return d * d;
    }
    return 1.0;
}

// complex Helmholtz kernel with equal quadrature weights: exp(i kappa r) / (n r),
// kappa = ell; coinciding points give 0
__device__ inline void kernel_gc(double ell, double npts, const double *a, const double *b, double &re, double &im) {
    const double dx = a[0] - b[0], dy = a[1] - b[1], dz = a[2] - b[2];
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    if (r == 0.0) {
        re = im = 0.0;
        return;
    }
    const double f = 1.0 / (npts * r);
    re = cos(ell * r) * f;
    im = sin(ell * r) * f;
}

// one-dimensional Lagrange polynomial j of the nodes nd[0..p) at x
__device__ inline double lagrange1(const double *nd, int p, int j, double x) {
    double v = 1.0, xj = nd[j];
    for (int i = 0; i < p; ++i) {
        if (i == j) continue;
        v *= (x - nd[i]) / (xj - nd[i]);
    }
    return v;
}

// tensor nodes: nu = jx + p*jy + p^2*jz, first-kind Chebyshev points of the box
__global__ void k_nodes(int32_t C, int p, const double *__restrict__ box, double *__restrict__ nodes) {
    const int k = p * p * p;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)C * k) return;
    const int32_t c = (int32_t)(idx / k);
    const int nu = (int)(idx % k);
    const int jj[3] = {nu % p, (nu / p) % p, nu / (p * p)};
    for (int d = 0; d < 3; ++d) {
        double lo = box[6 * c + d], hi = box[6 * c + 3 + d];
        double ctr = 0.5 * (lo + hi), half = 0.5 * (hi - lo);
        nodes[idx * 3 + d] = ctr + half * cos((2.0 * jj[d] + 1.0) * M_PI / (2.0 * p));
    }
}

__device__ inline void nodes1d(const double *nodes, int32_t c, int p, int d, double *nd) {
    const int k = p * p * p;
    const int stride = d == 0 ? 1 : (d == 1 ? p : p * p);
    for (int j = 0; j < p; ++j) nd[j] = nodes[((int64_t)c * k + (int64_t)j * stride) * 3 + d];
}

// V_t[i, nu] = L_{t,jx}(x_i) L_{t,jy}(y_i) L_{t,jz}(z_i) for the leaf t (one block per leaf)
template <typename T>
__global__ void k_fill_V(int p, const int32_t *__restrict__ leaves, const int32_t *__restrict__ first,
                         const int32_t *__restrict__ size, const double *__restrict__ pts,
                         const double *__restrict__ nodes, T *__restrict__ V, T *__restrict__ Vt,
                         const int64_t *__restrict__ vt_off) {
    const int k = p * p * p;
    const int32_t t = leaves[blockIdx.x];
    __shared__ double nd[3][16];
    if (threadIdx.x < 3 * p) {
        int d = threadIdx.x / p, j = threadIdx.x % p;
        const int stride = d == 0 ? 1 : (d == 1 ? p : p * p);
        nd[d][j] = nodes[((int64_t)t * k + (int64_t)j * stride) * 3 + d];
    }
    __syncthreads();
    const int64_t rows = size[t];
    for (int64_t e = threadIdx.x; e < rows * k; e += blockDim.x) {
        const int64_t i = first[t] + e / k;
        const int nu = (int)(e % k);
        const double *x = &pts[3 * i];
        double v = lagrange1(nd[0], p, nu % p, x[0]) * lagrange1(nd[1], p, (nu / p) % p, x[1]) *
                   lagrange1(nd[2], p, nu / (p * p), x[2]);
        V[i * k + nu] = from_double<T>(v);
        if (Vt) {
            // transposed copy: k x nt2 (rows padded to pad_rows(|t|), padding zero)
            const int64_t nt2 = pad_rows(rows), il = i - first[t];
            T *vt = Vt + vt_off[blockIdx.x];
            vt[nu * nt2 + il] = from_double<T>(v);
            if (il == rows - 1)
                for (int64_t z = rows; z < nt2; ++z) vt[nu * nt2 + z] = from_double<T>(0.0);
        }
    }
}

// E_c[a, nu] = L_{parent(c), nu}(xi_{c, a}) (one block per non-root cluster)
template <typename T>
__global__ void k_fill_E(int p, const int32_t *__restrict__ parent, const double *__restrict__ nodes,
                         T *__restrict__ E) {
    const int k = p * p * p;
    const int32_t c = blockIdx.x + 1;  // the root has no transfer matrix
    const int32_t par = parent[c];
    if (par < 0) {  // the root of a later system of a merged plan: zeros
        for (int e = threadIdx.x; e < k * k; e += blockDim.x) E[(int64_t)c * k * k + e] = from_double<T>(0.0);
        return;
    }
    __shared__ double nd[3][16];
    if (threadIdx.x < 3 * p) {
        int d = threadIdx.x / p, j = threadIdx.x % p;
        const int stride = d == 0 ? 1 : (d == 1 ? p : p * p);
        nd[d][j] = nodes[((int64_t)par * k + (int64_t)j * stride) * 3 + d];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < k * k; e += blockDim.x) {
        const int a = e / k, nu = e % k;
        const double *x = &nodes[((int64_t)c * k + a) * 3];
        double v = lagrange1(nd[0], p, nu % p, x[0]) * lagrange1(nd[1], p, (nu / p) % p, x[1]) *
                   lagrange1(nd[2], p, nu / (p * p), x[2]);
        E[(int64_t)c * k * k + e] = from_double<T>(v);
    }
}

// one-dimensional factors of the transfer matrices: F1[c][d][p i + j] = the father's j-th
// Lagrange polynomial on axis d at the son's i-th node on axis d, so that E_c[a, nu] =
// F1[c][0][a0, nu0] F1[c][1][a1, nu1] F1[c][2][a2, nu2] (digits a = a0 + p a1 + p^2 a2); the
// entries of a root (of every system of a merged plan) are zero
__global__ void k_fill_E1(int32_t C, int p, const int32_t *__restrict__ parent, const double *__restrict__ nodes,
                          double *__restrict__ F1) {
    const int per = 3 * p * p;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)C * per) return;
    const int32_t c = (int32_t)(idx / per);
    const int e = (int)(idx % per), d = e / (p * p), i = (e / p) % p, j = e % p;
    if (parent[c] < 0) {
        F1[idx] = 0.0;
        return;
    }
    double ndp[16], ndc[16];
    nodes1d(nodes, parent[c], p, d, ndp);
    nodes1d(nodes, c, p, d, ndc);
    F1[idx] = lagrange1(ndp, p, j, ndc[i]);
}

// S_b[nu, mu] = g(xi_{t,nu}, xi_{s,mu}), stored in the layout the coupling kernel reads
// (complex kernel: real part into S, imaginary part into S + s_plane)
template <typename T>
__global__ void k_fill_S(int k, int kernel, double ell, double npts, const int32_t *__restrict__ adm_row,
                         const int32_t *__restrict__ adm_col, const double *__restrict__ nodes,
                         T *__restrict__ S, int swz, int64_t s_blk, int64_t s_plane) {
    const int64_t b = blockIdx.x;
    const int32_t t = adm_row[b], s = adm_col[b];
    for (int e = threadIdx.x; e < k * k; e += blockDim.x) {
        const int nu = e / k, mu = e % k;
        const double *xa = &nodes[((int64_t)t * k + nu) * 3], *xb = &nodes[((int64_t)s * k + mu) * 3];
        const int64_t at = b * s_blk + s_index(swz, k, nu, mu);
        if (kernel == H2X_KERNEL_HELMHOLTZ) {
            double re, im;
            kernel_gc(ell, npts, xa, xb, re, im);
            S[at] = from_double<T>(re);
            S[at + s_plane] = from_double<T>(im);
        } else {
            S[at] = from_double<T>(kernel_g(kernel, ell, xa, xb));
        }
    }
    if (s_blk > k * k)  // the padding of layout 1
        for (int e = threadIdx.x; e < s_blk; e += blockDim.x) {
            int nu, mu;
            s_coords(swz, k, e, nu, mu);
            if (nu >= k || mu >= k) S[b * s_blk + e] = from_double<T>(0.0);
        }
}

// exp(-sqrt(r2) / ell), ie = 1 / ell.  The square root by Goldschmidt's iteration from the
// hardware's reciprocal square root, the quotient by a product and one correction; squared
// distances and length scales near the ends of the range take the library's forms.
__device__ inline double exp_kernel(double r2, double ell, double ie) {
    const double y = __builtin_amdgcn_rsq(r2);
    double g = r2 * y, h = 0.5 * y;
    const double e0 = fma(-h, g, 0.5);
    g = fma(g, e0, g);
    h = fma(h, e0, h);
    const double e1 = fma(-h, g, 0.5);
    g = fma(g, e1, g);
    h = fma(h, e1, h);
    g = fma(fma(-g, g, r2), h, g);
    if (!(r2 > 1e-280 && r2 < 1e280)) g = sqrt(r2);
    double q;
    if (ell > 1e-290 && ell < 1e290) {
        q = fmin(g * ie, 1e5);  // finite (and already beyond the exponential's range)
        q = fma(fma(-q, ell, g), ie, q);
    } else {
        q = g / ell;
    }
    return exp(-q);
}

// k_fill_S for the exponential kernel of order P, one work-group per block, in storage order (a
// 16-byte store per thread in the matrix-core layouts; padding entries are zero).  The nodes of a
// cluster are a tensor grid, so a squared distance is the sum of three entries of P x P tables
// of squared one-dimensional differences (LDS).  The kernel is symmetric: where the lists are
// (cptr given), the block (t, s) with t < s also writes the transposed block (s, t), entry i of
// column list t for entry i of row list t, and (s, t) writes nothing.  In layout 1 a thread then
// holds the 2 x 2 patch {nu, nu + 4} x {mu, mu + 4}, two 16-byte stores for either block.  In layout 0
// the transposed stores are single entries a row apart: blocks of orders 7 and 8 are evaluated
// each for itself (order 8, BF16, 30000 points: 7.2 ms from nodes, 11.2 with pairs, 5.3), and above
// order 4 the first two tables are summed in advance and the indices carried along, as the
// divisions by K and P cost more than the exponential (order 7, FP32: 0.98 -> 0.72 ms).
// P <= 2: launched with 64 threads, a thread per entry.
// Bound by the FP64 vector instructions of the square root and the exponential (about 65 an
// entry) and by the stores: 5.57 GB of rank-64 FP64 blocks in 1.10 ms (5.0 TB/s); 1.57 ms without
// the transposed blocks, 2.80 ms with nodes, divisions and 8-byte stores per entry.
template <typename T, int P>
__global__ __launch_bounds__(256) void k_fill_S_exp(double ell, const int32_t *__restrict__ adm_row,
                                                    const int32_t *__restrict__ adm_col,
                                                    const double *__restrict__ nodes, T *__restrict__ S, int64_t b0,
                                                    const int64_t *__restrict__ ptr, const int64_t *__restrict__ cptr,
                                                    const int64_t *__restrict__ cblk) {
    constexpr int K = P * P * P, KR = (K + 15) / 16 * 16, KC = (K + 7) / 8 * 8;
    constexpr int SWZ = K == 64 ? (sizeof(T) == 8 ? 1 : (sizeof(T) == 4 ? 2 : 3)) : (K > 64 && sizeof(T) == 8 ? 1 : 0);
    constexpr int G = SWZ ? 16 / (int)sizeof(T) : 1;
    constexpr int BLK = SWZ == 1 ? KR * KC : K * K;
    constexpr bool PATCH = SWZ == 1 && KR == KC;  // orders 4, 5 and 8
    constexpr bool LARGE0 = SWZ == 0 && P > 4;  // row-major and large: FP32 and BF16 above rank 64
    __shared__ double d2[3][P * P];
    __shared__ double d01[LARGE0 ? P * P * P * P : 1];  // the sums of the first two tables
    const int64_t b = b0 + blockIdx.x;
    const int32_t t = adm_row[b], s = adm_col[b];
    const bool pair = cptr && t != s && (PATCH || (SWZ == 0 && P <= 6));
    if (pair && t > s) return;
    const int tid = threadIdx.x;
    if (tid < 3 * P * P) {
        const int d = tid / (P * P), i = tid / P % P, j = tid % P, st = d == 0 ? 1 : (d == 1 ? P : P * P);
        const double v = nodes[((int64_t)t * K + i * st) * 3 + d] - nodes[((int64_t)s * K + j * st) * 3 + d];
        d2[d][i * P + j] = v * v;
    }
    __syncthreads();
    const double ie = 1.0 / ell;
    T *Sb = S + b * BLK, *Sp = pair ? S + cblk[cptr[t] + (b - ptr[t])] * BLK : nullptr;
    auto entry = [&](int nu, int mu) {
        const bool in = K % 16 == 0 || SWZ == 0 || (nu < K && mu < K);
        const int n1 = in ? nu : 0, m1 = in ? mu : 0;
        const double r2 = d2[1][n1 / P % P * P + m1 / P % P] + d2[0][n1 % P * P + m1 % P] +
                          d2[2][n1 / (P * P) * P + m1 / (P * P)];
        return in ? exp_kernel(r2, ell, ie) : 0.0;
    };
    if constexpr (PATCH) {
        typedef double dbl2 __attribute__((ext_vector_type(2)));
        constexpr int NPAT = KR * KC / 4, NU = (NPAT + 255) / 256;
#pragma unroll NU <= 4 ? NU : 2
        for (int u = 0; u < NU; ++u) {
            const int g = tid + 256 * u;
            if (NPAT % 256 != 0 && g >= NPAT) break;
            // patch g: rows nu, nu + 4 (8 a + 0..3 -> tile rows with bit 2 clear), columns mu, mu + 4
            const int r4 = g & 3, q = (g >> 2) & 3, ra = (g >> 4) % (KR / 8), ca = (g >> 4) / (KR / 8);
            const int nu = 8 * ra + r4, mu = 8 * ca + q;
            const double v00 = entry(nu, mu), v01 = entry(nu, mu + 4), v10 = entry(nu + 4, mu), v11 = entry(nu + 4, mu + 4);
            *(dbl2 *)(Sb + s_index(1, K, nu, mu)) = dbl2{v00, v01};
            *(dbl2 *)(Sb + s_index(1, K, nu + 4, mu)) = dbl2{v10, v11};
            if (pair) {
                *(dbl2 *)(Sp + s_index(1, K, mu, nu)) = dbl2{v00, v10};
                *(dbl2 *)(Sp + s_index(1, K, mu + 4, nu)) = dbl2{v01, v11};
            }
        }
    } else if constexpr (LARGE0) {
        constexpr int PP = P * P;
        for (int e = tid; e < PP * PP; e += 256) {
            const int n = e / PP, m = e % PP;
            d01[e] = d2[1][n / P * P + m / P] + d2[0][n % P * P + m % P];
        }
        __syncthreads();
        int nu = tid / K, mu = tid % K;
#pragma unroll 4
        for (int g = tid; g < BLK; g += 256) {
            const int n2 = nu / PP, m2 = mu / PP;
            const double r2 = d01[(nu - n2 * PP) * PP + mu - m2 * PP] + d2[2][n2 * P + m2];
            const T v = from_double<T>(exp_kernel(r2, ell, ie));
            Sb[g] = v;
            if (pair) Sp[mu * K + nu] = v;
            nu += 256 / K;
            mu += 256 % K;
            if (mu >= K) {
                mu -= K;
                ++nu;
            }
        }
    } else {
        constexpr int NU = (BLK / G + 255) / 256;
#pragma unroll NU <= 8 ? NU : 4
        for (int u = 0; u < NU; ++u) {
            const int g = tid + 256 * u;
            if (BLK / G % 256 != 0 && g >= BLK / G) break;
            T v[G];
#pragma unroll
            for (int x = 0; x < G; ++x) {
                int nu, mu;
                if constexpr (SWZ == 0) {
                    nu = g / K;
                    mu = g % K;
                } else if constexpr (SWZ == 1) {
                    const int lane = g & 63, rest = g >> 6;
                    nu = rest / (KC / 8) * 16 + (lane & 15);
                    mu = rest % (KC / 8) * 8 + 4 * x + (lane >> 4);
                } else {  // 4 G columns per chunk, G consecutive ones per lane
                    constexpr int NCH = K / (4 * G);
                    const int lane = g & 63, rest = g >> 6;
                    nu = rest / NCH * 16 + (lane & 15);
                    mu = rest % NCH * 4 * G + G * (lane >> 4) + x;
                }
                v[x] = from_double<T>(entry(nu, mu));
            }
            if constexpr (G == 1) {
                Sb[g] = v[0];
                if (pair) Sp[g % K * K + g / K] = v[0];
            } else {
                __builtin_memcpy(Sb + (int64_t)g * G, v, 16);
            }
        }
    }
}

// N_(t,s)[i, j] = g(x_i, x_j) + shift [i == j], row-major |t| x |s|, or stored
// transposed when trans != 0: |s| rows of length pad_rows(|t|), padding zero
// (complex kernel: real part into N, imaginary part into N + n_plane)
//
// One work-group per block, in tiles of up to 64 x 64 entries in storage order, so that the
// stores of a wave are consecutive.  Where the lists are symmetric (cptr given, real kernels),
// the block (t, s) with t < s also writes the block (s, t) out of an LDS tile: entry i of the
// column list of leaf t is the transposed block of entry i of its row list.
// Bound by the evaluation (about 130 vector instructions an entry) at four work-groups per CU:
// 1.2 GB of FP64 blocks of 43 points in 0.50 ms; 0.60 ms without the transposed blocks, 0.69 ms
// with 64-bit divisions and 8-byte stores a block row apart.
// TA: points per side of a tile: 64, or 32 or 16 (with 64 threads) where no leaf is larger.  A block of
// 8 points in a 64-wide tile took the LDS of a large one and 256 threads: refill of both S and N,
// n = 65536, leaves of 8, rank 1 0.40 ms before tiles, 0.60 with 64, 0.24 with 16; leaves of 16,
// rank 8 0.31 / 0.42 / 0.18; leaves of 24 0.28 / 0.33 / 0.28.
template <typename TN, int TA>
__global__ __launch_bounds__(TA > 16 ? 256 : 64) void k_fill_N(
                                                int kernel, double ell, double shift, double npts, int64_t q0,
                                                const int32_t *__restrict__ near_row,
                                                const int32_t *__restrict__ near_col,
                                                const int64_t *__restrict__ near_off,
                                                const int32_t *__restrict__ first, const int32_t *__restrict__ size,
                                                const double *__restrict__ pts, TN *__restrict__ N, int trans,
                                                int64_t n_plane, const int32_t *__restrict__ leaf_of,
                                                const int64_t *__restrict__ ptr, const int64_t *__restrict__ cptr,
                                                const int64_t *__restrict__ cblk) {
    constexpr int TL = TA, TH = TA > 16 ? 256 : 64;  // threads
    __shared__ TN tile[TL * (TA + 1)];
    __shared__ double pts_a[3][TA], pts_c[3][TL];  // the tile's points
    const int64_t q = q0 + blockIdx.x;
    const int32_t t = near_row[q], s = near_col[q];
    const bool cplx = kernel == H2X_KERNEL_HELMHOLTZ, sym = cptr && !cplx;
    if (sym && t > s) return;
    TN *Nb = N + near_off[q], *Np = nullptr;
    if (sym && t < s) {
        const int32_t l = leaf_of[t];
        Np = N + near_off[cblk[cptr[l] + (q - ptr[l])]];
    }
    // stored rows a (ra of them) of ca entries, padded to len: transposed, the points of s by those of t
    const int32_t ra = size[trans ? s : t], ca = size[trans ? t : s];
    const int32_t len = trans ? (int32_t)pad_rows(ca) : ca, lenp = trans ? (int32_t)pad_rows(ra) : ra;  // (lenp: of (s, t))
    const double *pa = pts + 3 * (int64_t)first[trans ? s : t], *pc = pts + 3 * (int64_t)first[trans ? t : s];
    const double ie = 1.0 / ell;
    for (int32_t a0 = 0; a0 < ra; a0 += TA)
        for (int32_t c0 = 0; c0 < ca; c0 += TL) {
            const int na = min(TA, ra - a0), nc = min(TL, ca - c0);
            const int dg = t == s ? c0 - a0 : 1 << 30;  // a - c on the diagonal
            TN *Na = Nb + (int64_t)a0 * len + c0;
            const float inv = 1.0f / (float)nc;
            if ((int)threadIdx.x < 3 * na) pts_a[threadIdx.x % 3][threadIdx.x / 3] = pa[3 * (int64_t)a0 + threadIdx.x];
            if ((int)threadIdx.x < 3 * nc) pts_c[threadIdx.x % 3][threadIdx.x / 3] = pc[3 * (int64_t)c0 + threadIdx.x];
            __syncthreads();
            for (int e = threadIdx.x; e < na * nc; e += TH) {
                const int a = (int)((e + 0.5f) * inv), c = e - a * nc;  // exact for e < 4096
                const double x[3] = {pts_c[0][c], pts_c[1][c], pts_c[2][c]};
                const double y[3] = {pts_a[0][a], pts_a[1][a], pts_a[2][a]};
                const int64_t at = (int64_t)a * len + c;
                const bool diag = a - c == dg;
                if (cplx) {
                    double re, im;
                    kernel_gc(ell, npts, x, y, re, im);
                    Na[at] = (TN)(diag ? re + shift : re);
                    Na[at + n_plane] = (TN)im;
                    continue;
                }
                double v;
                if (kernel == H2X_KERNEL_EXP) {
                    const double dx = x[0] - y[0], dy = x[1] - y[1], dz = x[2] - y[2];
                    v = exp_kernel(dx * dx + dy * dy + dz * dz, ell, ie);
                } else {
                    v = kernel_g(kernel, ell, x, y);
                }
                if (diag) v += shift;
                Na[at] = (TN)v;
                if (Np) tile[c * (TA + 1) + a] = (TN)v;
            }
            __syncthreads();
            if (!Np) continue;
            const float invp = 1.0f / (float)na;
            for (int e = threadIdx.x; e < na * nc; e += TH) {
                const int c = (int)((e + 0.5f) * invp), a = e - c * na;
                Np[(int64_t)(c0 + c) * lenp + a0 + a] = tile[c * (TA + 1) + a];
            }
            __syncthreads();
        }
    // padding
    if (len > ca)
        for (int32_t a = threadIdx.x; a < ra; a += TH) {
            Nb[(int64_t)a * len + ca] = (TN)0;
            if (cplx) Nb[(int64_t)a * len + ca + n_plane] = (TN)0;
        }
    if (Np && lenp > ra)
        for (int32_t c = threadIdx.x; c < ca; c += TH) Np[(int64_t)c * lenp + ra] = (TN)0;
}

// coupling matrices and near field, system by system (each with its own kernel
// parameters; a one-system operator uses the operator's current ones)
template <typename T, typename TN>
hipError_t fill_SN(const DevMat &dm, hipStream_t st) {
    const Plan &P = *dm.plan;
    const int32_t ns = P.nsys();
    for (int32_t i = 0; i < ns; ++i) {
        const int kernel = ns == 1 ? dm.kernel : (int)P.sys_prm[i].kernel;
        const double ell = ns == 1 ? dm.ell : P.sys_prm[i].ell, shift = ns == 1 ? dm.shift : P.sys_prm[i].shift;
        const int64_t a = P.sys_adm[i], na = P.sys_adm[i + 1] - a;
        const int64_t q = P.sys_near[i], nq = P.sys_near[i + 1] - q;
        const double npts = (double)(P.sys_row[i + 1] - P.sys_row[i]);  // points of system i
        // the exponential kernel in its own form per order
        auto fill_exp = [&](auto Pc) {
            constexpr int P1 = decltype(Pc)::value;
            hipLaunchKernelGGL((k_fill_S_exp<T, P1>), dim3((unsigned)na), dim3(P1 <= 2 ? 64 : 256), 0, st, ell,
                               dm.adm_row, dm.adm_col, dm.nodes, (T *)dm.S, a, dm.adm_ptr,
                               P.sym_lists ? dm.adm_cptr : nullptr, dm.adm_cblk);
        };
        if (na > 0 && kernel == H2X_KERNEL_EXP)
            switch (dm.p) {
                case 1: fill_exp(std::integral_constant<int, 1>{}); break;
                case 2: fill_exp(std::integral_constant<int, 2>{}); break;
                case 3: fill_exp(std::integral_constant<int, 3>{}); break;
                case 4: fill_exp(std::integral_constant<int, 4>{}); break;
                case 5: fill_exp(std::integral_constant<int, 5>{}); break;
                case 6: fill_exp(std::integral_constant<int, 6>{}); break;
                case 7: fill_exp(std::integral_constant<int, 7>{}); break;
                default: fill_exp(std::integral_constant<int, 8>{}); break;
            }
        else if (na > 0)
            hipLaunchKernelGGL(k_fill_S<T>, dim3((unsigned)na), dim3(256), 0, st, dm.k, kernel, ell, npts,
                               dm.adm_row + a, dm.adm_col + a, dm.nodes, (T *)dm.S + a * dm.s_blk, dm.swz, dm.s_blk,
                               dm.s_plane);
        auto fill_near = [&](auto TAc) {
            constexpr int TA = decltype(TAc)::value;
            hipLaunchKernelGGL((k_fill_N<TN, TA>), dim3((unsigned)nq), dim3(TA > 16 ? 256 : 64), 0, st, kernel, ell, shift,
                               npts, q, dm.near_row, dm.near_col, dm.near_off, dm.first, dm.size, dm.pts, (TN *)dm.N,
                               dm.near_t, dm.n_plane, dm.leaf_of, dm.near_ptr, P.sym_lists ? dm.near_cptr : nullptr,
                               dm.near_cblk);
        };
        if (nq > 0) {
            if (dm.max_leaf <= 16) fill_near(std::integral_constant<int, 16>{});
            else if (dm.max_leaf <= 32) fill_near(std::integral_constant<int, 32>{});
            else fill_near(std::integral_constant<int, 64>{});
        }
    }
    return hipGetLastError();
}

template <typename T, typename TN>
hipError_t fill_typed(const DevMat &dm, hipStream_t st) {
    const int64_t ck = (int64_t)dm.C * dm.k;
    hipLaunchKernelGGL(k_nodes, dim3((unsigned)((ck + 255) / 256)), dim3(256), 0, st, dm.C, dm.p, dm.box, dm.nodes);
    if (dm.L > 0)
        hipLaunchKernelGGL(k_fill_V<T>, dim3(dm.L), dim3(256), 0, st, dm.p, dm.leaves, dm.first, dm.size, dm.pts,
                           dm.nodes, (T *)dm.V, (T *)dm.Vt, dm.vt_off);
    if (dm.C > 1) {
        if (dm.E)
            hipLaunchKernelGGL(k_fill_E<T>, dim3(dm.C - 1), dim3(256), 0, st, dm.p, dm.parent, dm.nodes, (T *)dm.E);
        const int64_t nf = (int64_t)dm.C * 3 * dm.p * dm.p;
        hipLaunchKernelGGL(k_fill_E1, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, st, dm.C, dm.p, dm.parent,
                           dm.nodes, dm.E1);
    }
    return fill_SN<T, TN>(dm, st);
}

template <typename T, typename TN>
hipError_t refill_typed(const DevMat &dm, hipStream_t st) {
    return fill_SN<T, TN>(dm, st);
}

}  // namespace

hipError_t refill_ell(DevMat &dm, double ell, hipStream_t st) {
    dm.ell = ell;
    switch (dm.storage) {
        case H2X_F64: return refill_typed<double, double>(dm, st);
        case H2X_F32: return refill_typed<float, float>(dm, st);
        default: return refill_typed<bf16_t, float>(dm, st);
    }
}

size_t mat_layout(const Plan &P, h2x_prec storage, DevMat *dm, char *base) {
    size_t cur = 0;
    const int32_t C = P.C, L = (int32_t)P.leaves.size(), k = P.k;
    const int64_t n = P.n, na = (int64_t)P.adm_col.size(), nn = (int64_t)P.near_col.size();
    DevMat d;
    d.n = n; d.C = C; d.L = L; d.k = k; d.p = P.p; d.depth_max = P.depth_max; d.max_leaf = P.max_leaf;
    d.max_near_rows = P.max_near_rows;
    d.leaf_half = P.leaf_half;
    d.n_adm = na; d.n_near = nn; d.near_entries = P.near_entries; d.storage = storage;
    d.kernel = P.prm.kernel; d.ell = P.prm.ell; d.shift = P.prm.shift; d.plan = &P;
    // higher ranks of the FP64 operator (p = 5 to 8): their own matrix-core kernels
    d.gk = (storage == H2X_F64 && k > 64) ? 1 : 0;
    d.swz = d.gk ? 1 : (k != 64 ? 0 : (storage == H2X_F64 ? 1 : (storage == H2X_F32 ? 2 : 3)));
    d.s_blk = s_block(d.swz, k);
    // matrix-core layout (transposed near field, transposed leaf bases): FP64, k = 64 or k <= 32
    d.mc = (storage == H2X_F64 && (k == 64 || k <= 32)) ? 1 : 0;
    // low-precision operators with k = 64 use the same transposed near field (FP32) and leaf bases
    d.near_t = (d.mc || d.gk || (storage != H2X_F64 && (k == 64 || k <= 32))) ? 1 : 0;
    d.first = carve<int32_t>(cur, base, C);
    d.size = carve<int32_t>(cur, base, C);
    d.parent = carve<int32_t>(cur, base, C);
    d.son0 = carve<int32_t>(cur, base, C);
    d.son1 = carve<int32_t>(cur, base, C);
    d.leaves = carve<int32_t>(cur, base, L);
    d.lvl_all = carve<int32_t>(cur, base, C);
    d.lvl_inner = carve<int32_t>(cur, base, P.lvl_inner.size() + 1);
    d.up_son = carve<int32_t>(cur, base, 2 * P.lvl_inner.size() + 1);
    d.dn_par = carve<int32_t>(cur, base, C);
    d.up_rng = carve<int32_t>(cur, base, 4 * P.lvl_inner.size() + 1);
    d.dn_rng = carve<int32_t>(cur, base, 4 * (size_t)C);
    d.adm_ptr = carve<int64_t>(cur, base, C + 1);
    d.adm_col = carve<int32_t>(cur, base, na + 1);
    d.adm_row = carve<int32_t>(cur, base, na + 1);
    d.cpl_order = carve<int32_t>(cur, base, C);
    d.leaf_order = carve<int32_t>(cur, base, L);
    d.split_depth = P.split_depth;
    d.n_deep = (int32_t)P.cpl_deep.size();
    d.n_shallow = (int32_t)P.cpl_shallow.size();
    d.cpl_deep = carve<int32_t>(cur, base, d.n_deep + 1);
    d.cpl_shallow = carve<int32_t>(cur, base, d.n_shallow + 1);
    d.near_ptr = carve<int64_t>(cur, base, L + 1);
    d.near_col = carve<int32_t>(cur, base, nn + 1);
    d.near_row = carve<int32_t>(cur, base, nn + 1);
    d.near_off = carve<int64_t>(cur, base, nn + 1);
    d.vt_off = carve<int64_t>(cur, base, L + 1);
    d.near_off_rm = carve<int64_t>(cur, base, nn + 1);
    d.adm_cptr = carve<int64_t>(cur, base, C + 1);
    d.adm_cblk = carve<int64_t>(cur, base, na + 1);
    d.near_cptr = carve<int64_t>(cur, base, L + 1);
    d.near_cblk = carve<int64_t>(cur, base, nn + 1);
    d.sys_of = carve<int32_t>(cur, base, C);
    d.depth = carve<int32_t>(cur, base, C);
    d.leaf_of = carve<int32_t>(cur, base, C);
    d.perm = carve<int64_t>(cur, base, n);
    d.pts = carve<double>(cur, base, 3 * n);
    d.box = carve<double>(cur, base, 6 * (size_t)C);
    d.nodes = carve<double>(cur, base, 3 * (size_t)C * k);
    const size_t es = storage == H2X_F64 ? 8 : (storage == H2X_F32 ? 4 : 2);
    const size_t ens = storage == H2X_F64 ? 8 : 4;
    d.V = carve<char>(cur, base, es * (size_t)n * k);
    // (the transfer passes of the higher FP64 ranks read the one-dimensional factors only)
    d.E = d.gk ? nullptr : carve<char>(cur, base, es * (size_t)C * k * k);
    d.E1 = carve<double>(cur, base, 3 * (size_t)C * P.p * P.p);
    // complex kernel: a real and an imaginary plane of S and N (V and E stay real)
    d.cplx = (P.nsys() == 1 && P.prm.kernel == H2X_KERNEL_HELMHOLTZ) ? 1 : 0;
    const int planes = d.cplx ? 2 : 1;
    const int64_t nstored = d.near_t ? P.near_entries_t : P.near_entries;
    d.s_plane = d.cplx ? na * k * k : 0;
    d.n_plane = d.cplx ? nstored : 0;
    d.S = carve<char>(cur, base, es * planes * (size_t)(na ? na : 1) * d.s_blk);
    d.N = carve<char>(cur, base, ens * planes * (size_t)(nstored ? nstored : 1) + 16);
    d.Vt = d.near_t ? carve<char>(cur, base, es * (size_t)P.vt_entries) : nullptr;
    if (dm) *dm = d;
    return align_up(cur);
}

hipError_t launch_fill(const DevMat &dm, hipStream_t st) {
    switch (dm.storage) {
        case H2X_F64: return fill_typed<double, double>(dm, st);
        case H2X_F32: return fill_typed<float, float>(dm, st);
        default: return fill_typed<bf16_t, float>(dm, st);
    }
}

}  // namespace h2x
