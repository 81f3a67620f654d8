// Augmented operator for dense constraint rows (eq. augsys): at n = 200 the two
// streaming passes over the packed rows take 121 us, and everything else is
// small enough that the number of launches counts.  While script-A script-Q is
// small too (dense_explicit), the off-diagonal blocks are products with the
// explicit matrix (11.5 MB each way at n = 200, m = 2400, the matrices that the
// preconditioner uses), taken by the same launch as the last pass, so the operator
// is six launches (three for n <= 64) instead of sixteen: n = 200 182 -> 150 us, n =
// 20 41 -> 13 us.
#include "dense_op.hpp"

#include <hip/hip_ext.h>

#include "wave.hpp"

namespace wc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

// ---- E Y E and its packing for n <= 64, one workgroup ----------------------------
// Latency-bound: one launch instead of the partial sums, two products of one
// output tile each and the packing.  The eight waves share the (n / 16)^2 tiles
// of each product; the operands sit in LDS, zero padded to whole tiles.
constexpr int DM_T = 512;

__global__ __launch_bounds__(DM_T) void dense_mid_kernel(int n, int N2, int ldp, int nparts,
                                                         const double* __restrict__ part, long pstride,
                                                         const int* __restrict__ pj, const int* __restrict__ pk,
                                                         const double* __restrict__ E, double* __restrict__ mw) {
    extern __shared__ double dm[];
    const int nt = (n + 15) / 16, np = 16 * nt, pitch = np + 1;
    double* Ys = dm;                 // column-major, later M
    double* Es = Ys + np * pitch;
    double* Ts = Es + np * pitch;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    for (int t = tid; t < np * np; t += DM_T) {
        const int i = t % np, j = t / np;
        const bool in = i < n && j < n;
        Es[j * pitch + i] = in ? E[i + j * n] : 0.0;
        if (!in) Ys[j * pitch + i] = 0.0;
    }
    for (int p = tid; p < N2; p += DM_T) {
        double s = 0.0;
        int q = 0;
        for (; q + 4 <= nparts; q += 4) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = part[(q + u) * pstride + p];
#pragma unroll
            for (int u = 0; u < 4; ++u) s += x[u];
        }
        for (; q < nparts; ++q) s += part[q * pstride + p];
        const int j = pj[p], k = pk[p];
        Ys[j + k * pitch] = s;
        Ys[k + j * pitch] = s;
    }
    __syncthreads();
    auto product = [&](const double* A, const double* B, double* C) {
        for (int t = wave; t < nt * nt; t += DM_T / 64) {
            const int r0 = (t % nt) * 16, c0 = (t / nt) * 16;
            d4 a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};
            for (int k0 = 0; k0 < np; k0 += 8) {
                a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(k0 + lk) * pitch + r0 + li], B[(c0 + li) * pitch + k0 + lk],
                                                          a0, 0, 0, 0);
                a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(k0 + 4 + lk) * pitch + r0 + li],
                                                          B[(c0 + li) * pitch + k0 + 4 + lk], a1, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) C[(c0 + li) * pitch + r0 + lk + 4 * v] = a0[v] + a1[v];
        }
        __syncthreads();
    };
    product(Ys, Es, Ts);
    product(Es, Ts, Ys);
    for (int p = tid; p < ldp; p += DM_T) {
        double v = 0.0;
        if (p < N2) {
            const int j = pj[p], k = pk[p];
            v = (j == k) ? Ys[j + j * pitch] : Ys[j + k * pitch] + Ys[k + j * pitch];
        }
        mw[p] = v;
    }
}

void dense_mid(hipStream_t st, int n, long N2, long ldp, int nparts, const double* part, long pstride, const int* pj,
               const int* pk, const double* E, double* mw) {
    require(n >= 1 && n <= DENSE_MID_N, "dense_mid: n out of range");
    const int np = 16 * ((n + 15) / 16);
    hipLaunchKernelGGL(dense_mid_kernel, dim3(1), dim3(DM_T), 3 * sizeof(double) * np * (np + 1), st, n,
                       static_cast<int>(N2), static_cast<int>(ldp), nparts, part, pstride, pj, pk, E, mw);
    WC_LAUNCH_CHECK();
}

// ---- packing the split-K sum of E (Y E) -------------------------------------------
// The sum over the splits and the packing in one pass: the product itself is
// only ever read through its packed weights.
__global__ __launch_bounds__(256) void reduce_pack_kernel(int n, long N2, long ldp, int splits,
                                                          const double* __restrict__ P, const int* __restrict__ pj,
                                                          const int* __restrict__ pk, double* __restrict__ mw) {
    const long p = blockIdx.x * 256L + threadIdx.x;
    if (p >= ldp) return;
    double v = 0.0;
    if (p < N2) {
        const int j = pj[p], k = pk[p];
        const long nn = (long)n * n, o1 = j + (long)k * n, o2 = k + (long)j * n;
        double a = 0.0, b = 0.0;
        int s = 0;
        for (; s + 4 <= splits; s += 4) {
            double x[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = P[(s + u) * nn + o1];
                y[u] = P[(s + u) * nn + o2];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a += x[u];
                b += y[u];
            }
        }
        for (; s < splits; ++s) {
            a += P[s * nn + o1];
            b += P[s * nn + o2];
        }
        v = (j == k) ? a : a + b;
    }
    mw[p] = v;
}
void reduce_pack(hipStream_t st, int n, long N2, long ldp, int splits, const double* P, const int* pj, const int* pk,
                 double* mw) {
    hipLaunchKernelGGL(reduce_pack_kernel, dim3(cdiv(ldp, 256)), dim3(256), 0, st, n, N2, ldp, splits, P, pj, pk, mw);
    WC_LAUNCH_CHECK();
}

// ---- last pass ------------------------------------------------------------------------
// HBM-bound (the packed rows once).  The first workgroups take the d bottom
// rows, one per wave; the others two packed rows each, as packed_rows does,
// with the same rows' script-A script-Q products added before the reduction.
__device__ __forceinline__ double dot_piece(d2 a, const double* x) { return a.x * x[0] + a.y * x[1]; }

template <class T>
struct Piece;
template <>
struct Piece<double> {
    typedef d2 vec;
    static constexpr int W = 2, ROWS = 2;
    static __device__ __forceinline__ double dot(vec a, vec x) { return a.x * x.x + a.y * x.y; }
};
template <>
struct Piece<float> {
    typedef f4 vec;
    static constexpr int W = 4, ROWS = 4;
    static __device__ __forceinline__ double dot(vec a, vec x) {
        return (double)a.x * x.x + (double)a.y * x.y + (double)a.z * x.z + (double)a.w * x.w;
    }
};

template <class T>
__global__ __launch_bounds__(256) void op_rows_kernel(int m, int kw, const T* __restrict__ P, long ldp,
                                                      const T* __restrict__ mw, int d,
                                                      const double* __restrict__ AQ, long ldaq,
                                                      const double* __restrict__ AQt, long ldaqt,
                                                      const double* __restrict__ u, const double* __restrict__ v,
                                                      const double* __restrict__ sig, double t2,
                                                      double* __restrict__ out) {
    typedef typename Piece<T>::vec vec;
    constexpr int OP_ROWS = Piece<T>::ROWS;
    __shared__ double sh[4][OP_ROWS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nb = (d + 3) / 4;
    if (static_cast<int>(blockIdx.x) < nb) {
        const int c = blockIdx.x * 4 + wave;
        if (c >= d) return;  // whole waves leave
        const double* a = AQt + (long)c * ldaqt;
        double s0 = 0.0, s1 = 0.0;
        int i = 2 * lane;
        for (; i + 385 < m; i += 512) {
            d2 av[4];
            double x[4][2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                av[q] = *reinterpret_cast<const d2*>(a + i + 128 * q);
                x[q][0] = u[i + 128 * q];
                x[q][1] = u[i + 128 * q + 1];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q & 1) s1 += dot_piece(av[q], x[q]);
                else s0 += dot_piece(av[q], x[q]);
            }
        }
        for (; i < m; i += 128) {
            s0 += a[i] * u[i];
            if (i + 1 < m) s1 += a[i + 1] * u[i + 1];
        }
        const double s = wave_sum_all(s0 + s1);
        if (lane == 0) out[m + c] = s - t2 * sig[c] * v[c];
        return;
    }
    const int row0 = (blockIdx.x - nb) * OP_ROWS;
    double acc[OP_ROWS];
    const vec* prow[OP_ROWS];
    const double* arow[OP_ROWS];
#pragma unroll
    for (int r = 0; r < OP_ROWS; ++r) {
        const int row = row0 + r < m ? row0 + r : m - 1;
        prow[r] = reinterpret_cast<const vec*>(P + (long)row * ldp);
        arow[r] = AQ + (long)row * ldaq;
        acc[r] = 0.0;
    }
    const vec* x = reinterpret_cast<const vec*>(mw);
    for (int c = threadIdx.x; c < kw; c += 256) {
        const vec xv = x[c];
#pragma unroll
        for (int r = 0; r < OP_ROWS; ++r) acc[r] += Piece<T>::dot(__builtin_nontemporal_load(&prow[r][c]), xv);
    }
    for (int c = 2 * threadIdx.x; c < d; c += 512) {
        const double v0 = v[c], v1 = c + 1 < d ? v[c + 1] : 0.0;  // AQ rows are zero past d
#pragma unroll
        for (int r = 0; r < OP_ROWS; ++r) {
            const d2 a = *reinterpret_cast<const d2*>(arow[r] + c);
            acc[r] += a.x * v0 + a.y * v1;
        }
    }
#pragma unroll
    for (int r = 0; r < OP_ROWS; ++r) {
        const double s = wave_sum_all(acc[r]);
        if (lane == 0) sh[wave][r] = s;
    }
    __syncthreads();
    if (threadIdx.x < OP_ROWS && row0 + static_cast<int>(threadIdx.x) < m) {
        const int r = threadIdx.x;
        out[row0 + r] = (sh[0][r] + sh[1][r]) + (sh[2][r] + sh[3][r]);
    }
}

template <class T>
void op_rows(hipStream_t st, int m, long k, const T* P, long ldp, const T* mw, int d, const double* AQ, long ldaq,
             const double* AQt, long ldaqt, const double* u, const double* v, const double* sig, double t2,
             double* out, hipEvent_t t0, hipEvent_t t1) {
    constexpr int W = Piece<T>::W;
    require(ldp % W == 0 && ldaq % 2 == 0 && ldaqt % 2 == 0, "op_rows: row pitches must keep 16-byte alignment");
    const int kw = static_cast<int>(round_up(k, W) / W);
    hipExtLaunchKernelGGL(op_rows_kernel<T>, dim3(cdiv(d, 4) + cdiv(m, Piece<T>::ROWS)), dim3(256), 0, st, t0, t1, 0, m, kw,
                          P, ldp, mw, d, AQ, ldaq, AQt, ldaqt, u, v, sig, t2, out);
    WC_LAUNCH_CHECK();
}
template void op_rows<double>(hipStream_t, int, long, const double*, long, const double*, int, const double*, long,
                              const double*, long, const double*, const double*, const double*, double, double*,
                              hipEvent_t, hipEvent_t);
template void op_rows<float>(hipStream_t, int, long, const float*, long, const float*, int, const double*, long,
                             const double*, long, const double*, const double*, const double*, double, double*,
                             hipEvent_t, hipEvent_t);

// ---- preconditioner ---------------------------------------------------------------------
// At n = 200 AQ is 11.5 MB and stays in the caches, so a pass costs about its
// launch and one round of loads: the vector updates around each product ride
// along, and the two transposed products of the refinement share a pass (eight
// launches instead of seventeen, with the C^{-1} products).  Down passes: a
// workgroup per row of AQt (d rows of m); up passes: a wave per row of AQ.
template <int NX>
__device__ __forceinline__ void down_dots(int m, const double* __restrict__ a, const double* const (&x)[NX],
                                          double (&s)[NX]) {
    const d2* a2 = reinterpret_cast<const d2*>(a);
    const int m2 = (m + 1) / 2;
#pragma unroll
    for (int k = 0; k < NX; ++k) s[k] = 0.0;
    int c = threadIdx.x;
    for (; c + 768 < m2; c += 1024) {
        d2 av[4], xv[4][NX];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            av[q] = a2[c + 256 * q];
#pragma unroll
            for (int k = 0; k < NX; ++k) xv[q][k] = reinterpret_cast<const d2*>(x[k])[c + 256 * q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < NX; ++k) s[k] += av[q].x * xv[q][k].x + av[q].y * xv[q][k].y;
    }
    for (; c < m2; c += 256) {
        const d2 av = a2[c];
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const d2 xv = reinterpret_cast<const d2*>(x[k])[c];
            s[k] += av.x * xv.x + av.y * xv.y;
        }
    }
    __shared__ double sh[4][NX];
#pragma unroll
    for (int k = 0; k < NX; ++k) {
        const double t = wave_sum_all(s[k]);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NX; ++k) s[k] = (sh[0][k] + sh[1][k]) + (sh[2][k] + sh[3][k]);
}

__global__ __launch_bounds__(256) void precond_down_kernel(int m, const double* __restrict__ AQt, long ldaqt,
                                                           const double* __restrict__ f, const double* __restrict__ h,
                                                           double ib, double* __restrict__ td) {
    const int c = blockIdx.x;
    const double* const x[1] = {f};
    double s[1];
    down_dots<1>(m, AQt + (long)c * ldaqt, x, s);
    if (threadIdx.x == 0) td[c] = h[c] - ib * s[0];
}
__global__ __launch_bounds__(256) void precond_down2_kernel(int m, const double* __restrict__ AQt, long ldaqt,
                                                            const double* __restrict__ z1,
                                                            const double* __restrict__ rho,
                                                            const double* __restrict__ h,
                                                            const double* __restrict__ sig, double t2,
                                                            const double* __restrict__ zv, double ib,
                                                            double* __restrict__ td) {
    const int c = blockIdx.x;
    const double* const x[2] = {z1, rho};
    double s[2];
    down_dots<2>(m, AQt + (long)c * ldaqt, x, s);
    if (threadIdx.x == 0) td[c] = (h[c] - s[0] + t2 * sig[c] * zv[c]) - ib * s[1];
}
void precond_down(hipStream_t st, int m, int d, const double* AQt, long ldaqt, const double* f, const double* h,
                  double ib, double* td) {
    hipLaunchKernelGGL(precond_down_kernel, dim3(d), dim3(256), 0, st, m, AQt, ldaqt, f, h, ib, td);
    WC_LAUNCH_CHECK();
}
void precond_down2(hipStream_t st, int m, int d, const double* AQt, long ldaqt, const double* z1, const double* rho,
                   const double* h, const double* sig, double t2, const double* zv, double ib, double* td) {
    hipLaunchKernelGGL(precond_down2_kernel, dim3(d), dim3(256), 0, st, m, AQt, ldaqt, z1, rho, h, sig, t2, zv, ib,
                       td);
    WC_LAUNCH_CHECK();
}

// AQ_i . x by one wave, delivered to all its lanes
__device__ __forceinline__ double up_dot(int d, const double* __restrict__ a, const double* __restrict__ x) {
    const d2* a2 = reinterpret_cast<const d2*>(a);
    const d2* x2 = reinterpret_cast<const d2*>(x);
    const int lane = threadIdx.x & 63, k2 = (d + 1) / 2;
    double s0 = 0.0, s1 = 0.0;
    int c = lane;
    for (; c + 192 < k2; c += 256) {
        d2 av[4], xv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            av[u] = a2[c + 64 * u];
            xv[u] = x2[c + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double t = av[u].x * xv[u].x + av[u].y * xv[u].y;
            if (u & 1) s1 += t;
            else s0 += t;
        }
    }
    for (; c < k2; c += 64) s0 += a2[c].x * x2[c].x + a2[c].y * x2[c].y;
    return wave_sum_all(s0 + s1);
}
__global__ __launch_bounds__(256) void precond_up_kernel(int m, int d, const double* __restrict__ AQ, long ldaq,
                                                         const double* __restrict__ zv, const double* __restrict__ f,
                                                         double ib, double beta, double* __restrict__ z1,
                                                         double* __restrict__ rho) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= m) return;  // whole waves leave
    const double t = up_dot(d, AQ + (long)i * ldaq, zv);
    if ((threadIdx.x & 63) == 0) {
        const double fi = f[i];
        const double z = ib * fi + (-ib) * t;
        z1[i] = z;
        rho[i] = (-beta) * z + (fi - t);
    }
}
__global__ __launch_bounds__(256) void precond_up2_kernel(int m, int d, const double* __restrict__ AQ, long ldaq,
                                                          const double* __restrict__ zv,
                                                          const double* __restrict__ zv2,
                                                          const double* __restrict__ rho, double ib,
                                                          double* __restrict__ z1, double* __restrict__ zout) {
    const int nb = (m + 3) / 4;
    if (static_cast<int>(blockIdx.x) >= nb) {
        const int c = (blockIdx.x - nb) * 256 + threadIdx.x;
        if (c < d) zout[c] = zv[c] + zv2[c];
        return;
    }
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= m) return;
    const double t = up_dot(d, AQ + (long)i * ldaq, zv2);
    if ((threadIdx.x & 63) == 0) z1[i] = (ib * rho[i] + (-ib) * t) + z1[i];
}
void precond_up(hipStream_t st, int m, int d, const double* AQ, long ldaq, const double* zv, const double* f, double ib,
                double beta, double* z1, double* rho) {
    hipLaunchKernelGGL(precond_up_kernel, dim3(cdiv(m, 4)), dim3(256), 0, st, m, d, AQ, ldaq, zv, f, ib, beta, z1, rho);
    WC_LAUNCH_CHECK();
}
void precond_up2(hipStream_t st, int m, int d, const double* AQ, long ldaq, const double* zv, const double* zv2,
                 const double* rho, double ib, double* z1, double* zout) {
    hipLaunchKernelGGL(precond_up2_kernel, dim3(cdiv(m, 4) + cdiv(d, 256)), dim3(256), 0, st, m, d, AQ, ldaq, zv, zv2,
                       rho, ib, z1, zout);
    WC_LAUNCH_CHECK();
}

}  // namespace wc
