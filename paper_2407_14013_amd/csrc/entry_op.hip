// Entry-sampling script-A script-Q products (Section 6).  For A_i = sym(e_j e_k^T)
//   (AQ v)_i = (U_j . q_k + U_k . q_j) / 2 with U = G_w H(v), and
//   (AQ)^T u = [svec; sqrt2 vec] of F = G_w^T (A^T(u) Q),
// H = [B; sqrt2 N] and q_j the first r entries of row j of G_w.  While G_w is
// small every piece is a few microseconds of latency, so each product is two
// launches with the coordinate maps and the vector updates inside (n = 301, m =
// 9000: 14 us to 7 us for AQ v, 16 to 8 us for (AQ)^T u); past that the two passes
// over G_w are bound by its bytes, and the refinement's two transposed products
// share one.
#include "entry_op.hpp"

#include "launch_plan.hpp"
#include "sdp_kernels.hpp"
#include "wave.hpp"

namespace wc {

constexpr double kS2 = 1.4142135623730951;
constexpr double kIS2 = 0.7071067811865476;

// svec position c (0-based) of an r x r symmetric block -> (row i, column jj), i >= jj
__device__ inline void svec_ij(int c, int r, int& i, int& jj) {
    jj = 0;
    while (c >= r - jj) {
        c -= r - jj;
        ++jj;
    }
    i = jj + c;
}
// entry (a, b) of H(v)
__device__ inline double h_entry(const double* v, int n, int r, int a, int b) {
    if (a < r) {
        const int i = a > b ? a : b, jj = a > b ? b : a;
        const int c = jj * r - jj * (jj - 1) / 2 + (i - jj);
        return (i == jj) ? v[c] : v[c] * kIS2;
    }
    return kS2 * v[r * (r + 1) / 2 + (a - r) + (long)(n - r) * b];
}

// ---- YQ = A^T(u) Q, row by row ------------------------------------------------------
// One wave per row; four entries per lane in flight (their indices, then the
// gathers), NV vectors at once.  R >= r columns.
template <int R, int NV>
__global__ __launch_bounds__(256) void entry_yq2_kernel(int n, int r, const int* __restrict__ rptr,
                                                        const int* __restrict__ rcol, const int* __restrict__ ridx,
                                                        const double* __restrict__ u0, const double* __restrict__ u1,
                                                        const double* __restrict__ Q, double* __restrict__ YQ) {
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= n) return;  // whole waves leave together
    double acc[NV][R];
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int b = 0; b < R; ++b) acc[k][b] = 0.0;
    const int e0 = rptr[j], e1 = rptr[j + 1];
    constexpr int EU = R <= 4 ? 4 : 1;
    for (int e = e0 + lane; e < e1; e += 64 * EU) {
        int p[EU], i[EU];
#pragma unroll
        for (int x = 0; x < EU; ++x) {
            const int ee = min(e + 64 * x, e1 - 1);
            p[x] = rcol[ee];
            i[x] = ridx[ee];
        }
        double w[EU][NV], q[EU][R];
#pragma unroll
        for (int x = 0; x < EU; ++x) {
            const bool in = e + 64 * x < e1;
            const double w0 = u0[i[x]];
            w[x][0] = in ? w0 : 0.0;
            if constexpr (NV > 1) {
                const double w1 = u1[i[x]];
                w[x][1] = in ? w1 : 0.0;
            }
#pragma unroll
            for (int b = 0; b < R; ++b) q[x][b] = b < r ? Q[p[x] + (long)b * n] : 0.0;
        }
#pragma unroll
        for (int x = 0; x < EU; ++x) {
            const double f = p[x] == j ? 1.0 : 0.5;
#pragma unroll
            for (int k = 0; k < NV; ++k)
#pragma unroll
                for (int b = 0; b < R; ++b) acc[k][b] += f * w[x][k] * q[x][b];
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int b = 0; b < R; ++b) {
            if (b >= r) break;
            const double v = wave_sum_all(acc[k][b]);
            if (lane == 0) YQ[j + (long)(k * r + b) * n] = v;
        }
}

// ---- F = G_w^T YQ read in v-coordinates ---------------------------------------------
// out[c] = a0 F0(c) + a1 F1(c) + add[c] + ts sig[c] vin[c].
struct VOut {
    double a0, a1, ts;
    const double *add, *sig, *vin;
    double* out;
};
__device__ inline void v_put(const VOut& o, int c, double f0, double f1) {
    double v = o.a0 * f0;
    if (o.a1 != 0.0) v += o.a1 * f1;
    if (o.add != nullptr) v += o.add[c];
    if (o.vin != nullptr) v += o.ts * o.sig[c] * o.vin[c];
    o.out[c] = v;
}

// column T_k of B dotted with u
__device__ inline double lp_col(const EntryLp& lp, int k, const double* u) {
    double s = 0.0;
    for (int q = lp.cptr[lp.Tl[k]]; q < lp.cptr[lp.Tl[k] + 1]; ++q) s += lp.cval[q] * u[lp.crow[q]];
    return s;
}
// the LP entries of out, d .. d + t - 1
__device__ inline void lp_put(const EntryLp& lp, const VOut& o, int d, int k, const double* u0, const double* u1) {
    if (k < lp.t) v_put(o, d + k, lp_col(lp, k, u0), u1 != nullptr ? lp_col(lp, k, u1) : 0.0);
}
// row i of B[:, T] dotted with the LP entries vlp
__device__ inline double lp_row(const EntryLp& lp, int i, const double* vlp) {
    double s = 0.0;
    if (lp.t > 0)
        for (int q = lp.rptr[i]; q < lp.rptr[i + 1]; ++q) {
            const int p = lp.pos[lp.rcol[q]];
            if (p >= 0) s += lp.rval[q] * vlp[p];
        }
    return s;
}

// Small n: one wave per row a >= r of F (a contiguous column of G_w); the first
// workgroup takes the r top rows, whose symmetric part svec needs.
template <int R, int NV>
__global__ __launch_bounds__(256) void entry_fv_kernel(int n, int r, const double* __restrict__ Gw,
                                                       const double* __restrict__ YQ, VOut o, EntryLp lp,
                                                       const double* __restrict__ u0,
                                                       const double* __restrict__ u1) {
    __shared__ double top[NV][EN_R][EN_R];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc[NV][R];
    auto row = [&](int a) {
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int b = 0; b < R; ++b) acc[k][b] = 0.0;
        const double* g = Gw + (long)a * n;
        constexpr int U = R <= 4 ? 4 : 1;
        for (int i = lane; i < n; i += 64 * U) {
            double x[U], y[U][NV][R];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int ii = min(i + 64 * q, n - 1);
                const double gv = g[ii];
                x[q] = i + 64 * q < n ? gv : 0.0;
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int b = 0; b < R; ++b) y[q][k][b] = (b < r && i + 64 * q < n) ? YQ[ii + (long)(k * r + b) * n] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int b = 0; b < R; ++b) acc[k][b] += x[q] * y[q][k][b];
        }
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int b = 0; b < R; ++b)
                if (b < r) acc[k][b] = wave_sum_all(acc[k][b]);
    };
    const int nb = r * (r + 1) / 2;
    if (blockIdx.x == 0) {
        for (int a = wave; a < r; a += 4) {
            row(a);
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int b = 0; b < R; ++b)
                        if (b < r) top[k][a][b] = acc[k][b];
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < nb; c += 256) {
            int i, jj;
            svec_ij(c, r, i, jj);
            double f[2] = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < NV; ++k)
                f[k] = (i == jj) ? top[k][i][i] : kS2 * 0.5 * (top[k][i][jj] + top[k][jj][i]);
            v_put(o, c, f[0], f[1]);
        }
        return;
    }
    const int nrow = (n - r + 3) / 4;
    if (static_cast<int>(blockIdx.x) > nrow) {
        lp_put(lp, o, nb + (n - r) * r, (blockIdx.x - 1 - nrow) * 256 + threadIdx.x, u0, u1);
        return;
    }
    const int a = r + (blockIdx.x - 1) * 4 + wave;
    if (a >= n) return;
    row(a);
    // lane b writes column b's coordinate
    double f0 = 0.0, f1 = 0.0;
#pragma unroll
    for (int b = 0; b < R; ++b) {
        if (lane == b) {
            f0 = acc[0][b];
            if constexpr (NV > 1) f1 = acc[1][b];
        }
    }
    if (lane < r) v_put(o, nb + (a - r) + (n - r) * lane, kS2 * f0, kS2 * f1);
}

// Large n: F (ld n, the second vector's columns after the first's r) by the
// thin product, then its v-coordinates.
__global__ __launch_bounds__(256) void entry_f_to_v_kernel(int n, int r, const double* __restrict__ F, int nv, VOut o,
                                                           EntryLp lp, const double* __restrict__ u0,
                                                           const double* __restrict__ u1) {
    const int nb = r * (r + 1) / 2, d = nb + (n - r) * r;
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= d) {
        lp_put(lp, o, d, c - d, u0, u1);
        return;
    }
    double f[2] = {0.0, 0.0};
    for (int k = 0; k < nv; ++k) {
        const double* Fk = F + (long)k * r * n;
        if (c < nb) {
            int i, jj;
            svec_ij(c, r, i, jj);
            f[k] = (i == jj) ? Fk[i + (long)i * n] : kS2 * 0.5 * (Fk[i + (long)jj * n] + Fk[jj + (long)i * n]);
        } else {
            const int t = c - nb;
            f[k] = kS2 * Fk[(r + t % (n - r)) + (long)(t / (n - r)) * n];
        }
    }
    v_put(o, c, f[0], f[1]);
}

static int dim_v(const EntryAq& q) { return q.r * (q.r + 1) / 2 + (q.n - q.r) * q.r; }

template <int R, int NV>
static void yq_launch(hipStream_t st, const EntryAq& q, const double* u0, const double* u1, int r, const double* Q,
                      double* YQ) {
    hipLaunchKernelGGL((entry_yq2_kernel<R, NV>), dim3(cdiv(q.n, 4)), dim3(256), 0, st, q.n, r, q.rptr, q.rcol, q.ridx,
                       u0, u1, Q, YQ);
    WC_LAUNCH_CHECK();
}

void entry_aqt(hipStream_t st, const EntryAq& q, const double* u0, double a0, const double* u1, double a1,
               const double* add, double ts, const double* vin, double* out) {
    const int n = q.n, r = q.r, nv = u1 != nullptr ? 2 : 1, d = r * (r + 1) / 2 + (n - r) * r;
    const VOut o{a0, u1 != nullptr ? a1 : 0.0, ts, add, q.sig, vin, out};
    if (r <= 4) {
        if (nv == 2) yq_launch<4, 2>(st, q, u0, u1, r, q.Gw, q.YQ);
        else yq_launch<4, 1>(st, q, u0, nullptr, r, q.Gw, q.YQ);
    } else {
        for (int k = 0; k < nv; ++k)
            for (int b0 = 0; b0 < r; b0 += EN_R)  // EN_R columns of Q per launch
                yq_launch<EN_R, 1>(st, q, k ? u1 : u0, nullptr, std::min(EN_R, r - b0), q.Gw + (long)b0 * n,
                                   q.YQ + (long)(k * r + b0) * n);
    }
    if (entry_small(n, r)) {
        const dim3 grid(1 + cdiv(n - r, 4) + cdiv(q.lp.t, 256));
        if (r <= 4 && nv == 2)
            hipLaunchKernelGGL((entry_fv_kernel<4, 2>), grid, dim3(256), 0, st, n, r, q.Gw, q.YQ, o, q.lp, u0, u1);
        else if (r <= 4)
            hipLaunchKernelGGL((entry_fv_kernel<4, 1>), grid, dim3(256), 0, st, n, r, q.Gw, q.YQ, o, q.lp, u0, u1);
        else if (nv == 2)
            hipLaunchKernelGGL((entry_fv_kernel<EN_R, 2>), grid, dim3(256), 0, st, n, r, q.Gw, q.YQ, o, q.lp, u0, u1);
        else
            hipLaunchKernelGGL((entry_fv_kernel<EN_R, 1>), grid, dim3(256), 0, st, n, r, q.Gw, q.YQ, o, q.lp, u0, u1);
        WC_LAUNCH_CHECK();
        return;
    }
    const int per = thin_vectors(r, nv);
    for (int k = 0; k < nv; k += per)
        q.product(true, per * r, q.YQ + (long)k * r * n, q.F + (long)k * r * n);
    hipLaunchKernelGGL(entry_f_to_v_kernel, dim3(cdiv(d + q.lp.t, 256)), dim3(256), 0, st, n, r, q.F, nv, o,
                       q.lp, u0, u1);
    WC_LAUNCH_CHECK();
}

// ---- U = G_w H(v) ---------------------------------------------------------------------
// Small n: a workgroup owns 16 rows, its 16 thread groups a sixteenth of K
// each, H formed from v in LDS; eight loads of G_w in flight per thread.
template <int R>
__global__ __launch_bounds__(256) void entry_u_kernel(int n, int r, const double* __restrict__ Gw,
                                                      const double* __restrict__ v, double* __restrict__ U) {
    extern __shared__ double H[];  // n x r
    __shared__ double red[16][R][16];
    for (int b = 0; b < r; ++b)
#pragma unroll 4
        for (int a = threadIdx.x; a < n; a += 256) H[a + b * n] = h_entry(v, n, r, a, b);
    __syncthreads();
    const int li = threadIdx.x & 15, kg = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + li, ic = min(i, n - 1);
    double acc[R];
#pragma unroll
    for (int b = 0; b < R; ++b) acc[b] = 0.0;
    for (int k = kg; k < n; k += 128) {
        double g[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int kk = min(k + 16 * u, n - 1);
            const double x = Gw[ic + (long)kk * n];
            g[u] = k + 16 * u < n ? x : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (k + 16 * u < n) {
#pragma unroll
                for (int b = 0; b < R; ++b)
                    if (b < r) acc[b] += g[u] * H[k + 16 * u + b * n];
            }
        }
    }
#pragma unroll
    for (int b = 0; b < R; ++b) red[kg][b][li] = acc[b];
    __syncthreads();
    if (kg < r && i < n) {
        for (int b = kg; b < r; b += 16) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 16; ++q) s += red[q][b][li];
            U[i + (long)b * n] = s;
        }
    }
}

void entry_form_u(hipStream_t st, const EntryAq& q, const double* v) {
    const int n = q.n, r = q.r;
    if (entry_small(n, r)) {
        const size_t lds = sizeof(double) * (size_t)n * r;
        if (r <= 4)
            hipLaunchKernelGGL(entry_u_kernel<4>, dim3(cdiv(n, 16)), dim3(256), lds, st, n, r, q.Gw, v, q.U);
        else
            hipLaunchKernelGGL(entry_u_kernel<EN_R>, dim3(cdiv(n, 16)), dim3(256), lds, st, n, r, q.Gw, v, q.U);
        WC_LAUNCH_CHECK();
        return;
    }
    v_to_h(st, n, r, v, q.Hm);
    q.product(false, r, q.Hm, q.U);
}

// (U_j . q_k + U_k . q_j) / 2
__device__ inline double aq_entry(int n, int r, int j, int k, const double* __restrict__ U,
                                  const double* __restrict__ Q) {
    double s = 0.0;
    int b = 0;
    for (; b + 2 <= r; b += 2) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const long o = (long)(b + u) * n;
            x[4 * u] = U[j + o];
            x[4 * u + 1] = Q[k + o];
            x[4 * u + 2] = U[k + o];
            x[4 * u + 3] = Q[j + o];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) s += x[4 * u] * x[4 * u + 1] + x[4 * u + 2] * x[4 * u + 3];
    }
    for (; b < r; ++b) s += U[j + (long)b * n] * Q[k + (long)b * n] + U[k + (long)b * n] * Q[j + (long)b * n];
    return 0.5 * s;
}

__global__ __launch_bounds__(256) void entry_aq_op_kernel(int m, int n, int r, const int* __restrict__ jk,
                                                          const double* __restrict__ U, const double* __restrict__ Q,
                                                          const double* __restrict__ M, int lower, int splits,
                                                          double* __restrict__ out) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const int j = jk[2 * i], k = jk[2 * i + 1];  // j <= k
    double g;
    if (M == nullptr) {
        g = out[i];
    } else if (splits > 0) {
        const long nn = (long)n * n, o1 = j + (long)k * n, o2 = k + (long)j * n;
        double a = 0.0, b = 0.0;
        int s = 0;
        for (; s + 4 <= splits; s += 4) {
            double x[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = M[(s + u) * nn + o1];
                y[u] = M[(s + u) * nn + o2];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a += x[u];
                b += y[u];
            }
        }
        for (; s < splits; ++s) {
            a += M[s * nn + o1];
            b += M[s * nn + o2];
        }
        g = 0.5 * (a + b);
    } else if (lower) {
        g = M[k + (long)j * n];
    } else {
        g = 0.5 * (M[j + (long)k * n] + M[k + (long)j * n]);
    }
    out[i] = g + aq_entry(n, r, j, k, U, Q);
}
__global__ __launch_bounds__(256) void entry_aq_up_kernel(int m, int n, int r, const int* __restrict__ jk,
                                                          const double* __restrict__ U, const double* __restrict__ Q,
                                                          const double* __restrict__ f, double ib, double beta,
                                                          double* __restrict__ z1, double* __restrict__ rho,
                                                          EntryLp lp, const double* __restrict__ vlp) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const double t = aq_entry(n, r, jk[2 * i], jk[2 * i + 1], U, Q) + lp_row(lp, i, vlp), fi = f[i];
    const double z = ib * fi + (-ib) * t;
    z1[i] = z;
    rho[i] = (-beta) * z + (fi - t);
}
__global__ __launch_bounds__(256) void entry_aq_up2_kernel(int m, int n, int r, const int* __restrict__ jk,
                                                           const double* __restrict__ U, const double* __restrict__ Q,
                                                           const double* __restrict__ rho, double ib,
                                                           double* __restrict__ z1, int d,
                                                           const double* __restrict__ zv,
                                                           const double* __restrict__ zv2, double* __restrict__ zout,
                                                           EntryLp lp, const double* __restrict__ vlp) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < m) {
        const double t = aq_entry(n, r, jk[2 * i], jk[2 * i + 1], U, Q) + lp_row(lp, i, vlp);
        z1[i] = (ib * rho[i] + (-ib) * t) + z1[i];
    } else if (i < m + d) {
        zout[i - m] = zv[i - m] + zv2[i - m];
    }
}

void entry_aq_op(hipStream_t st, const EntryAq& q, const double* M, bool lower, int splits, double* out) {
    hipLaunchKernelGGL(entry_aq_op_kernel, dim3(cdiv(q.m, 256)), dim3(256), 0, st, q.m, q.n, q.r, q.jk, q.U, q.Gw, M,
                       lower ? 1 : 0, splits, out);
    WC_LAUNCH_CHECK();
}
void entry_aq_up(hipStream_t st, const EntryAq& q, const double* v, const double* f, double ib, double beta, double* z1,
                 double* rho) {
    entry_form_u(st, q, v);
    hipLaunchKernelGGL(entry_aq_up_kernel, dim3(cdiv(q.m, 256)), dim3(256), 0, st, q.m, q.n, q.r, q.jk, q.U, q.Gw, f,
                       ib, beta, z1, rho, q.lp, v + dim_v(q));
    WC_LAUNCH_CHECK();
}
void entry_aq_up2(hipStream_t st, const EntryAq& q, const double* v, const double* rho, double ib, double* z1,
                  const double* zv, double* zout) {
    entry_form_u(st, q, v);
    const int d = dim_v(q) + q.lp.t;
    hipLaunchKernelGGL(entry_aq_up2_kernel, dim3(cdiv((long)q.m + d, 256)), dim3(256), 0, st, q.m, q.n, q.r, q.jk, q.U,
                       q.Gw, rho, ib, z1, d, zv, v, zout, q.lp, v + dim_v(q));
    WC_LAUNCH_CHECK();
}

}  // namespace wc
