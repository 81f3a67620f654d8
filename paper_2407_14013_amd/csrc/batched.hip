// Many small, uneven SDPs solved in one persistent launch.
//
// Every workgroup (512 threads) takes instances from an atomic queue, largest
// first, and runs the whole interior-point method of solver.hip for one
// instance at a time: the Nesterov-Todd scaling (Introduction, eq. newt), its
// eigen-split and the reformulated Newton system (Section 3, eq. EQSigdef and
// eq. augsys), indefinite PCG with the Section 6 preconditioner (Corollary
// pcg), recovery (eq. recover) and the Mehrotra predictor-corrector step.  All
// dense linear algebra is done by the workgroup on matrices in its own global
// scratch (n <= 128, so they stay in L2): matrix-core GEMMs with the operands
// read straight from cache, unblocked Cholesky, Gauss-Jordan sweeps for the
// SPD inverse of the preconditioner's Schur complement, one-sided (Hestenes)
// Jacobi for the SVD and the eigen-decomposition, Lanczos with multisection
// for step lengths.  The constraint data (packed rows) is streamed by the two
// passes of the augmented operator.  Every workgroup reaches the queue's end,
// so the grid always drains.
//
// One workgroup alone on its CU is bound by latency: a Krylov iteration is a
// chain of phases, each a round of loads, sums and a barrier.  So every loop
// here issues a batch of loads (clamped indices, no serial tail) before it
// uses them, products that share their operand share a pass (pcg_t), sums stay
// in the vector pipeline (wave.hpp), the Krylov vectors live in LDS, and each
// phase is a function of its own that reads the pointers it needs from LDS
// (held in scalar registers over the whole method they spilled at every use,
// and untyped they made every access a flat one).  256 instances with n in
// [16, 24]: 1 120 ms with 256 threads and one load or one product per phase,
// 210 to 250 ms in this form; one instance of n = 24, m = 216: 242 to 54 us per
// Krylov iteration, all else included; n = 128, m = 1152: 16.0 to 2.8 s per solve.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <exception>
#include <numeric>
#include <type_traits>
#include <vector>

#include "batched.hpp"
#include "host_pool.hpp"
#include "launch_plan.hpp"
#include "sdp_kernels.hpp"
#include "wave.hpp"

namespace wc {
namespace {

constexpr int BT = 512;           // threads per workgroup
constexpr int BWV = BT / 64;      // waves per workgroup
constexpr int BLZ = 64;           // Lanczos steps at most
constexpr double kS2 = 1.4142135623730951;
constexpr double kIS2 = 0.7071067811865476;

struct BInst {
    int n, m, rmax, rows_per_wave, aq_group, gemm_tile;
    long N2, ldp, ldp32;
    const double* P;  // m x ldp packed rows
    const float* P32; // m x ldp32 packed rows rounded to FP32 (low-precision inner solves), else null
    const double* b;
    const double* C;  // n x n
    double xi, eta, mean_a2, bnorm, Cnorm;
    double* Xout;
    double* yout;
};

struct BOut {
    int status, iterations;
    long long pcg, matvecs, lp_matvecs;
    double pobj, dobj, relgap, pinf, dinf, mu;
};

struct BParams {
    int nmax, mmax, dmax, rcap;
    long N2max;
    long per_wg;  // doubles of scratch per workgroup
    double inner_tol, gap_tol, feas_tol, step_frac;
    int inner_maxit, max_ipm_iter;
    int lowp;           // FP32 inner operator with FP64 refinement sweeps
    int max_refine;
    double refine_tol;  // residual reduction asked of each low-precision PCG run
};

// ---------------------------------------------------------------------------
// Workgroup primitives.  Every one ends with a barrier, so consecutive calls
// see each other's results; all threads call them with the same arguments.
// Pointers carry their address space (gd: global scratch, ld: LDS), so that
// loads are global or LDS instructions also where a function is not inlined.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(1))) double gd;
typedef __attribute__((address_space(1))) int gi;
typedef __attribute__((address_space(1))) float gf;
typedef __attribute__((address_space(3))) double ld;
typedef __attribute__((address_space(3))) int li;

__device__ __forceinline__ void bsync() { __syncthreads(); }

__device__ __forceinline__ double wg_sum(double v, ld* red) {
    v = wave_sum_all(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    bsync();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < BWV; ++i) s += red[i];
    bsync();
    return s;
}

__device__ __forceinline__ double wg_max(double v, ld* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    bsync();
    double s = red[0];
#pragma unroll
    for (int i = 1; i < BWV; ++i) s = fmax(s, red[i]);
    bsync();
    return s;
}

template <class X, class Y>
__device__ __forceinline__ double wg_dot(int n, X x, Y y, ld* red) {
    double a = 0.0;
    for (int t = threadIdx.x; t < n; t += BT) a += x[t] * y[t];
    return wg_sum(a, red);
}

template <class X>
__device__ __forceinline__ void wg_fill(int n, X x, double v) {
    for (int t = threadIdx.x; t < n; t += BT) x[t] = v;
    bsync();
}
template <class X, class Y>
__device__ __forceinline__ void wg_copy(int n, X x, Y y) {
    for (int t = threadIdx.x; t < n; t += BT) y[t] = x[t];
    bsync();
}
// z = a x + b y (z may alias x or y)
__device__ __forceinline__ void wg_axpby(int n, double a, const gd* x, double b, const gd* y, gd* z) {
    for (int t = threadIdx.x; t < n; t += BT) z[t] = a * x[t] + b * y[t];
    bsync();
}
__device__ __noinline__ void wg_symmetrize(int n, gd* A) {
    for (int t = threadIdx.x; t < n * n; t += BT) {
        const int i = t % n, j = t / n;
        if (i > j) {
            const double v = 0.5 * (A[i + j * n] + A[j + i * n]);
            A[i + j * n] = v;
            A[j + i * n] = v;
        }
    }
    bsync();
}
__device__ __forceinline__ void wg_identity(int n, gd* A, double v) {
    for (int t = threadIdx.x; t < n * n; t += BT) A[t] = (t % n == t / n) ? v : 0.0;
    bsync();
}
__device__ __forceinline__ void wg_transpose(int n, const gd* A, gd* B) {
    for (int t = threadIdx.x; t < n * n; t += BT) {
        const int i = t % n, j = t / n;
        B[j + i * n] = A[t];
    }
    bsync();
}
// s^pw for the powers used: 1, 1/2, -1/2
__device__ __forceinline__ double half_pow(double s, double pw) {
    return pw == 1.0 ? s : (pw > 0.0 ? sqrt(s) : 1.0 / sqrt(s));
}
// B(:, k) = A(:, k) * s[k]^pw
__device__ __forceinline__ void wg_scale_cols(int rows, int cols, const gd* A, const gd* s, double pw, gd* B) {
    for (int t = threadIdx.x; t < rows * cols; t += BT) B[t] = A[t] * half_pow(s[t / rows], pw);
    bsync();
}
// B(k, :) = A(k, :) * s[k]^pw
__device__ __forceinline__ void wg_scale_rows(int n, const gd* A, const gd* s, double pw, gd* B) {
    for (int t = threadIdx.x; t < n * n; t += BT) B[t] = A[t] * half_pow(s[t % n], pw);
    bsync();
}

// Wave tile edge of the workgroup's MFMA products for the instance it is
// solving (16 or 32, the instance's gemm_tile), set at the start of each instance.
__shared__ int wg_tile;

// C = alpha op(A) op(B) + beta C, column-major, with T = double on the FP64
// matrix cores (16x16x4) or T = float on the FP32 ones (the FP64 operands
// rounded as they are read, FP32 accumulation, C in FP64).  Each wave computes
// TS x TS output tiles (TS = 32: 2 x 2 blocks; TS = 16: one, so that small
// products keep more of the workgroup's waves busy) with the operands read
// straight from cache: lane l supplies A[l % 16][l / 16], B[l / 16][l % 16];
// accumulator element v of lane l is D[l / 16 + 4 v][l % 16] in FP64 and
// D[4 (l / 16) + v][l % 16] in FP32.  A product is bound by the latency of its
// loads, so a step takes 16 or 32 of K (all its loads in flight, unconditional: the
// indices are clamped and A zeroed past K) and the next step's loads are
// issued before this one's matrix instructions.  C must not alias A or B.
template <class T> struct Acc4;
template <> struct Acc4<double> { typedef double v __attribute__((ext_vector_type(4))); };
template <> struct Acc4<float> { typedef float v __attribute__((ext_vector_type(4))); };

template <class T, int TS>
__device__ __forceinline__ void wg_gemm_t(bool ta, bool tb, int M, int N, int K, double alpha, const gd* A, int lda,
                                          const gd* B, int ldb, double beta, gd* C, int ldc) {
    constexpr int NB = TS / 16, KS = TS == 16 ? 8 : 4;  // K per step: 32 or 16
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int tm = (M + TS - 1) / TS, tn = (N + TS - 1) / TS;
    const int sai = ta ? lda : 1, sak = ta ? 1 : lda, sbj = tb ? 1 : ldb, sbk = tb ? ldb : 1;
    for (int t = wave; t < tm * tn; t += BWV) {
        const int r0 = (t % tm) * TS, c0 = (t / tm) * TS;
        typename Acc4<T>::v acc[NB][NB];
        long ia[NB], jb[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            ia[x] = (long)min(r0 + x * 16 + li, M - 1) * sai;
            jb[x] = (long)min(c0 + x * 16 + li, N - 1) * sbj;
#pragma unroll
            for (int y = 0; y < NB; ++y) acc[x][y] = typename Acc4<T>::v{0, 0, 0, 0};
        }
        T a[KS][NB], bb[KS][NB];
        auto load = [&](int k0) {
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                const int k = k0 + 4 * u + lk, kc = min(k, K - 1);
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    const double v = A[ia[x] + (long)kc * sak];
                    a[u][x] = static_cast<T>(k < K ? v : 0.0);
                    bb[u][x] = static_cast<T>(B[jb[x] + (long)kc * sbk]);
                }
            }
        };
        load(0);
        for (int k0 = 0; k0 < K; k0 += 4 * KS) {
            T ca[KS][NB], cb[KS][NB];
#pragma unroll
            for (int u = 0; u < KS; ++u)
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    ca[u][x] = a[u][x];
                    cb[u][x] = bb[u][x];
                }
            if (k0 + 4 * KS < K) load(k0 + 4 * KS);
#pragma unroll
            for (int u = 0; u < KS; ++u)
#pragma unroll
                for (int x = 0; x < NB; ++x)
#pragma unroll
                    for (int y = 0; y < NB; ++y) {
                        if constexpr (sizeof(T) == 8)
                            acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[u][x], cb[u][y], acc[x][y], 0, 0, 0);
                        else
                            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[u][x], cb[u][y], acc[x][y], 0, 0, 0);
                    }
        }
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = r0 + x * 16 + (sizeof(T) == 8 ? lk + 4 * v : 4 * lk + v);
                    const int j = c0 + y * 16 + li;
                    if (i < M && j < N) {
                        gd* c = C + i + (long)j * ldc;
                        const double val = alpha * static_cast<double>(acc[x][y][v]);
                        *c = (beta == 0.0) ? val : val + beta * (*c);
                    }
                }
    }
    bsync();
}
// the general product (set-up of a Newton system, once or a few times each)
__device__ __noinline__ void wg_gemm(bool ta, bool tb, int M, int N, int K, double alpha, const gd* A, int lda,
                                     const gd* B, int ldb, double beta, gd* C, int ldc) {
    if (wg_tile == 16) wg_gemm_t<double, 16>(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
    else wg_gemm_t<double, 32>(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
}
// E Y E of the operator: T = Y E (E symmetric, read as its transpose, along its
// columns), then M = E T
template <class T>
__device__ __forceinline__ void wg_sandwich(int n, const gd* E, const gd* Y, gd* Tm, gd* M) {
    if (wg_tile == 16) {
        wg_gemm_t<T, 16>(false, true, n, n, n, 1.0, Y, n, E, n, 0.0, Tm, n);
        wg_gemm_t<T, 16>(false, false, n, n, n, 1.0, E, n, Tm, n, 0.0, M, n);
    } else {
        wg_gemm_t<T, 32>(false, true, n, n, n, 1.0, Y, n, E, n, 0.0, Tm, n);
        wg_gemm_t<T, 32>(false, false, n, n, n, 1.0, E, n, Tm, n, 0.0, M, n);
    }
}

// f(i, A_i . x) for every row i of a row-major A, by the 16 lanes that share
// the row (four rows per wave at a time, RB such batches in flight, eight
// columns per lane, indices clamped); f is called by all 16 lanes with the
// same sum.  No barrier.
template <class X, class F>
__device__ __forceinline__ void wg_rows(int rows, int cols, const gd* A, int lda, X x, F&& f) {
    constexpr int RB = 3;
    const int l = threadIdx.x & 15, slot = threadIdx.x >> 4;
    for (int i0 = 0; i0 < rows; i0 += RB * (BT / 16)) {
        double s[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) s[q] = 0.0;
        for (int c0 = l; c0 - l < cols; c0 += 128) {
            double av[RB][8], xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = c0 + 16 * u, cc = min(c, cols - 1);
#pragma unroll
                for (int q = 0; q < RB; ++q) av[q][u] = A[(long)min(i0 + q * (BT / 16) + slot, rows - 1) * lda + cc];
                const double v = x[cc];
                xv[u] = c < cols ? v : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int q = 0; q < RB; ++q) s[q] += av[q][u] * xv[u];
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int i = i0 + q * (BT / 16) + slot;
            const double t = row16_sum(s[q]);
            if (i < rows) f(i, t);
        }
    }
}

// f(c, A(:, c) . x) for every column c of a row-major A: one thread per
// column, eight rows in flight; with few columns the rows are split over
// groups of threads whose partial sums are added in order (part: BT doubles).
template <class X, class F>
__device__ __forceinline__ void wg_cols(int rows, int cols, const gd* A, int lda, X x, ld* part, F&& f) {
    auto span = [&](int c, int i0, int i1) {
        double s = 0.0;
        int i = i0;
        for (; i + 8 <= i1; i += 8) {
            double av[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) av[u] = A[(long)(i + u) * lda + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += av[u] * x[i + u];
        }
        for (; i < i1; ++i) s += A[(long)i * lda + c] * x[i];
        return s;
    };
    const int groups = cols < BT ? BT / cols : 1;
    if (groups > 1) {
        const int g = threadIdx.x / cols, c = threadIdx.x % cols, per = (rows + groups - 1) / groups;
        if (g < groups) part[threadIdx.x] = span(c, min(rows, g * per), min(rows, (g + 1) * per));
        bsync();
        for (int t = threadIdx.x; t < cols; t += BT) {
            double s = 0.0;
            for (int q = 0; q < groups; ++q) s += part[q * cols + t];
            f(t, s);
        }
    } else {
        for (int c = threadIdx.x; c < cols; c += BT) f(c, span(c, 0, rows));
    }
    bsync();
}

// In-place lower Cholesky; returns 0 or the 1-based index of the first
// non-positive pivot.  The strict upper triangle is set to zero.  A bad pivot
// also returns through a barrier: the caller may refill A at once, before a
// slower wave has read the pivot.
__device__ __noinline__ int wg_potrf(int n, gd* A, long lda) {
    for (int j = 0; j < n; ++j) {
        const double d = A[j + (long)j * lda];
        if (!(d > 0.0)) {  // every thread read the same value
            bsync();
            return j + 1;
        }
        const double s = sqrt(d);
        bsync();
        for (int i = j + 1 + threadIdx.x; i < n; i += BT) A[i + (long)j * lda] /= s;
        if (threadIdx.x == 0) A[j + (long)j * lda] = s;
        bsync();
        const int w = n - j - 1;
        for (int t = threadIdx.x; t < w * w; t += BT) {
            const int i = j + 1 + t % w, k = j + 1 + t / w;
            if (i >= k) A[i + (long)k * lda] -= A[i + (long)j * lda] * A[k + (long)j * lda];
        }
        bsync();
    }
    for (int t = threadIdx.x; t < n * n; t += BT) {
        const int i = t % n, j = t / n;
        if (i < j) A[i + (long)j * lda] = 0.0;
    }
    bsync();
    return 0;
}

// Linv = L^{-1} (lower): each thread forms whole columns by forward substitution.
__device__ __noinline__ void wg_trtri(int n, const gd* L, gd* Li) {
    for (int j = threadIdx.x; j < n; j += BT) {
        gd* x = Li + (long)j * n;
        for (int i = 0; i < j; ++i) x[i] = 0.0;
        x[j] = 1.0 / L[j + (long)j * n];
        for (int i = j + 1; i < n; ++i) {
            double s = 0.0;
            int k = j;
            for (; k + 4 <= i; k += 4) {
                double a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = L[i + (long)(k + u) * n];
                    b[u] = x[k + u];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) s += a[u] * b[u];
            }
            for (; k < i; ++k) s += L[i + (long)k * n] * x[k];
            x[i] = -s / L[i + (long)i * n];
        }
    }
    bsync();
}

// In-place inverse of a symmetric positive definite A (d x d, pitch lda) by
// Gauss-Jordan sweeps on every pivot (after all d sweeps A holds -A^{-1});
// returns 0 or the 1-based index of a non-positive pivot.  colk: d doubles.
// Wave w takes the columns w, w + 8, ..., its lanes the rows, four in flight.
__device__ __noinline__ int wg_spd_inverse(int d, gd* A, int lda, gd* colk) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = 0; k < d; ++k) {
        const double p = A[k + (long)k * lda];
        if (!(p > 0.0)) {
            bsync();
            return k + 1;
        }
        for (int i = threadIdx.x; i < d; i += BT) colk[i] = A[i + (long)k * lda];
        bsync();
        const double ip = 1.0 / p;
        for (int i = lane; i < d; i += 64) {
            const double ci = colk[i];
            for (int j0 = wave; j0 < d; j0 += 4 * BWV) {
                double av[4], cj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = min(j0 + u * BWV, d - 1);
                    av[u] = A[i + (long)j * lda];
                    cj[u] = colk[j];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u * BWV;
                    if (j < d) {
                        double v;
                        if (i == k && j == k) v = -ip;
                        else if (j == k) v = ci * ip;
                        else if (i == k) v = cj[u] * ip;
                        else v = av[u] - ci * cj[u] * ip;
                        A[i + (long)j * lda] = v;
                    }
                }
            }
        }
        bsync();
    }
    for (int j = wave; j < d; j += BWV)
        for (int i = lane; i < d; i += 64) A[i + (long)j * lda] = -A[i + (long)j * lda];
    bsync();
    return 0;
}

__device__ __forceinline__ void rr_pair(int round, int w, int N, int& a, int& b) {
    if (w == 0) {
        a = round;
        b = N - 1;
    } else {
        a = (round + w) % (N - 1);
        b = (round - w + (N - 1)) % (N - 1);
    }
}

// One-sided (Hestenes) Jacobi on the columns of A (n x n, pitch n), rotations
// accumulated in V (identity on entry).  Column pairs follow a round-robin
// tournament; each pair is handled by a group of tpp lanes of one wave.
// Afterwards sig[k] = ||A(:, k)|| in decreasing order and V's columns are
// permuted to match and signed so that each one's entry of largest magnitude
// is positive (lowest index on ties).  tmp: n x n scratch; ir: 2n ints.
__device__ __noinline__ int wg_jacobi(int n, gd* A, gd* V, gd* sig, gd* tmp, gd* nrm, gi* rank, double tol,
                         int max_sweeps, ld* red) {
    const int N = (n & 1) ? n + 1 : n;
    const int npairs = N / 2;
    int tpp = 64;
    while (tpp > 1 && tpp * npairs > BT) tpp >>= 1;
    const int groups = BT / tpp;
    const int g = threadIdx.x / tpp, li = threadIdx.x % tpp;
    int sweeps = 0;
    for (; sweeps < max_sweeps; ++sweeps) {
        double off = 0.0;
        for (int round = 0; round < N - 1; ++round) {
            for (int q0 = 0; q0 < npairs; q0 += groups) {
                const int q = q0 + g;
                int a = 0, b = 0;
                bool act = q < npairs;
                if (act) {
                    rr_pair(round, q, N, a, b);
                    act = a < n && b < n;
                }
                double al = 0.0, be = 0.0, ga = 0.0;
                if (act) {
                    const gd* ca = A + (long)a * n;
                    const gd* cb = A + (long)b * n;
                    for (int i = li; i < n; i += tpp) {
                        const double x = ca[i], y = cb[i];
                        al += x * x;
                        be += y * y;
                        ga += x * y;
                    }
                }
                // the lanes of a group are consecutive lanes of one wave
                for (int o = tpp / 2; o > 0; o >>= 1) {
                    al += __shfl_xor(al, o, 64);
                    be += __shfl_xor(be, o, 64);
                    ga += __shfl_xor(ga, o, 64);
                }
                if (act && fabs(ga) > tol * sqrt(al * be) && ga != 0.0) {
                    off = fmax(off, fabs(ga) / sqrt(al * be));
                    const double z = (be - al) / (2.0 * ga);
                    const double t = (z >= 0.0 ? 1.0 : -1.0) / (fabs(z) + sqrt(1.0 + z * z));
                    const double c = 1.0 / sqrt(1.0 + t * t), s = t * c;
                    gd* ca = A + (long)a * n;
                    gd* cb = A + (long)b * n;
                    gd* va = V + (long)a * n;
                    gd* vb = V + (long)b * n;
                    for (int i = li; i < n; i += tpp) {
                        const double x = ca[i], y = cb[i];
                        ca[i] = c * x - s * y;
                        cb[i] = s * x + c * y;
                        const double u = va[i], w = vb[i];
                        va[i] = c * u - s * w;
                        vb[i] = s * u + c * w;
                    }
                }
            }
            bsync();
        }
        if (wg_max(off, red) <= tol) {
            ++sweeps;
            break;
        }
    }
    // norms, ranks (decreasing, ties by index), signs, permutation
    for (int k = threadIdx.x; k < n; k += BT) {
        double s = 0.0, best = -1.0, bv = 1.0;
        for (int i = 0; i < n; ++i) {
            const double x = A[i + (long)k * n];
            s += x * x;
            const double v = V[i + (long)k * n];
            if (fabs(v) > best) {
                best = fabs(v);
                bv = v;
            }
        }
        nrm[k] = sqrt(s);
        nrm[n + k] = bv < 0.0 ? -1.0 : 1.0;
    }
    bsync();
    for (int k = threadIdx.x; k < n; k += BT) {
        int r = 0;
        for (int j = 0; j < n; ++j) r += (nrm[j] > nrm[k]) || (nrm[j] == nrm[k] && j < k);
        rank[k] = r;
    }
    bsync();
    for (int t = threadIdx.x; t < n * n; t += BT) {
        const int i = t % n, k = t / n;
        tmp[i + (long)rank[k] * n] = nrm[n + k] * V[t];
    }
    for (int k = threadIdx.x; k < n; k += BT) sig[rank[k]] = nrm[k];
    bsync();
    wg_copy(n * n, tmp, V);
    return sweeps;
}

// Number of eigenvalues below x of the tridiagonal (a, b), k x k.
__device__ __forceinline__ int sturm(const gd* a, const gd* b, int k, double x) {
    int cnt = 0;
    double d = 1.0;
    for (int i = 0; i < k; ++i) {
        const double bb = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
        d = a[i] - x - (i > 0 ? bb / d : 0.0);
        if (d == 0.0) d = -1e-300;
        if (d < 0.0) ++cnt;
    }
    return cnt;
}

// Smallest Ritz value of the symmetric T (n x n) after min(n, 64) Lanczos
// steps with full reorthogonalisation (twice), then multisection of the
// tridiagonal: every thread tests one point per round.
__device__ __noinline__ double wg_lanczos_min(int n, const gd* T, gd* Q, gd* w, gd* ab, ld* red, ld* h,
                                 li* ired) {
    const int kmax = n < BLZ ? n : BLZ;
    double loc = 0.0;
    for (int i = threadIdx.x; i < n; i += BT) {
        const double v = 1.0 + 0.5 * sin(1.0 + 0.7071067811865476 * i) + 0.25 * cos(0.3 * i * i);
        w[i] = v;
        loc += v * v;
    }
    const double nr0 = sqrt(wg_sum(loc, red));
    for (int i = threadIdx.x; i < n; i += BT) Q[i] = w[i] / nr0;
    bsync();
    double beta_prev = 0.0;
    int k = 0;
    for (int j = 0; j < kmax; ++j) {
        const gd* q = Q + (long)j * n;
        for (int i = threadIdx.x; i < n; i += BT) {
            double s = 0.0;
            for (int l = 0; l < n; ++l) s += T[i + (long)l * n] * q[l];
            w[i] = s;
        }
        bsync();
        const double alpha = wg_dot(n, q, w, red);
        for (int i = threadIdx.x; i < n; i += BT) {
            double v = w[i] - alpha * q[i];
            if (j > 0) v -= beta_prev * Q[i + (long)(j - 1) * n];
            w[i] = v;
        }
        bsync();
        for (int pass = 0; pass < 2; ++pass) {
            const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
            for (int l = wave; l <= j; l += BWV) {
                double s = 0.0;
                for (int i = lane; i < n; i += 64) s += Q[i + (long)l * n] * w[i];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
                if (lane == 0) h[l] = s;
            }
            bsync();
            for (int i = threadIdx.x; i < n; i += BT) {
                double v = w[i];
                for (int l = 0; l <= j; ++l) v -= h[l] * Q[i + (long)l * n];
                w[i] = v;
            }
            bsync();
        }
        const double beta = sqrt(wg_dot(n, w, w, red));
        if (threadIdx.x == 0) {
            ab[j] = alpha;
            ab[BLZ + j] = beta;
        }
        k = j + 1;
        if (!(beta > 1e-13 * (fabs(alpha) + beta_prev)) || j + 1 == kmax) break;
        for (int i = threadIdx.x; i < n; i += BT) Q[i + (long)(j + 1) * n] = w[i] / beta;
        beta_prev = beta;
        bsync();
    }
    bsync();
    // Gershgorin interval, then 8 rounds of (BT + 1)-way multisection
    double lo = ab[0], hi = ab[0];
    for (int i = 0; i < k; ++i) {
        const double rr = (i > 0 ? fabs(ab[BLZ + i - 1]) : 0.0) + (i + 1 < k ? fabs(ab[BLZ + i]) : 0.0);
        lo = fmin(lo, ab[i] - rr);
        hi = fmax(hi, ab[i] + rr);
    }
    for (int round = 0; round < 8; ++round) {
        const double step = (hi - lo) / (BT + 1);
        const double x = lo + (threadIdx.x + 1) * step;
        const int c = sturm(ab, ab + BLZ, k, x);
        if (threadIdx.x == 0) *ired = BT;
        bsync();
        if (c >= 1) atomicMin((int*)ired, static_cast<int>(threadIdx.x));
        bsync();
        const int t = *ired;
        bsync();
        const double nhi = (t < BT) ? lo + (t + 1) * step : hi;
        const double nlo = (t < BT) ? lo + t * step : lo + BT * step;
        lo = nlo;
        hi = nhi;
    }
    return 0.5 * (lo + hi);
}

// ---------------------------------------------------------------------------
// One instance.
// ---------------------------------------------------------------------------
struct Work {
    gd *X, *S, *L, *Linv, *R, *Rinv, *G, *Ginv, *Gw, *Gt, *E, *Y, *T1, *T2, *Mm, *Rd, *Ct, *dXa, *dSa, *dX, *dS,
        *Hc, *Vs, *Tp, *Q;
    gd *y, *rp, *dya, *dy, *tm, *lam, *dnt, *evE, *srt, *nrm, *sig, *U, *Hm, *YQ, *F;
    gd *vx, *vr, *vz, *vp, *vKp, *vg, *vtmp, *rho, *dz, *vres, *vdx, *td, *td2, *td3, *AQ, *Cm, *colk, *mw, *yp,
        *Taq, *ab;
    gi *pj, *pk, *rank;
    long ldaq;
};

__device__ __forceinline__ Work carve(gd* base, const BParams& bp) {
    Work w;
    gd* p = base;
    const long nn = (long)bp.nmax * bp.nmax;
    auto take = [&](long cnt) {
        gd* q = p;
        p += (cnt + 7) & ~7L;
        return q;
    };
    gd** mats[] = {&w.X,  &w.S,   &w.L,  &w.Linv, &w.R,   &w.Rinv, &w.G,  &w.Ginv, &w.Gw,
                       &w.Gt, &w.E,   &w.Y,  &w.T1,   &w.T2,  &w.Mm,   &w.Rd, &w.Ct,   &w.dXa,
                       &w.dSa, &w.dX, &w.dS, &w.Hc,   &w.Vs,  &w.Tp};
    for (gd** m : mats) *m = take(nn);
    w.Q = take((long)bp.nmax * (BLZ + 1));
    const long mv = bp.mmax + 8;
    w.y = take(mv);
    w.rp = take(mv);
    w.dya = take(mv);
    w.dy = take(mv);
    w.tm = take(mv);
    w.lam = take(bp.nmax);
    w.dnt = take(bp.nmax);
    w.evE = take(bp.nmax);
    w.srt = take(bp.nmax);
    w.nrm = take(2L * bp.nmax);
    w.sig = take(bp.dmax);
    const long nr = (long)bp.nmax * bp.rcap;
    w.U = take(nr);
    w.Hm = take(nr);
    w.YQ = take(nr);
    w.F = take(nr);
    const long NV = bp.mmax + bp.dmax + 8;
    gd** vecs[] = {&w.vx, &w.vr, &w.vz, &w.vp, &w.vKp, &w.vg, &w.vtmp, &w.rho, &w.dz, &w.vres, &w.vdx};
    for (gd** v : vecs) *v = take(NV);
    w.td = take(bp.dmax);
    w.td2 = take(bp.dmax);
    w.td3 = take(bp.dmax);
    w.ldaq = bp.dmax;
    w.AQ = take((long)bp.mmax * bp.dmax);
    w.Cm = take((long)bp.dmax * bp.dmax);
    w.colk = take(bp.dmax);
    w.mw = take(bp.N2max + 8);
    w.yp = take(bp.N2max + 8);
    w.Taq = take(16L * bp.nmax * bp.rcap);
    w.ab = take(2L * BLZ);
    w.pj = (gi*)(take(bp.N2max / 2 + 8));
    w.pk = (gi*)(take(bp.N2max / 2 + 8));
    w.rank = (gi*)(take(bp.nmax / 2 + 8));
    return w;
}

// The vectors of the Krylov loop (V: LDS or global pointers).  Each iteration
// passes over them in about fifteen phases of a few hundred cycles, so where
// they fit they live in LDS.
constexpr int PCG_KC = 16;  // columns per lane of the longest row that stays in registers: d <= 256
constexpr int PCG_PART = BWV * 2 * 16 * PCG_KC;  // doubles of cross-wave partial sums (>= 2 BT)
static_assert(PCG_PART >= 2 * BT, "the constraint pass keeps two partial sums per thread");

// Everything a phase needs, in LDS: the phases are functions of their own that
// read the few pointers and sizes they use from here (some sixty pointers held
// in scalar registers over the whole method spill at every use).
template <class V>
struct Inst {
    BInst I;
    BParams bp;
    Work w;
    ld* red;       // LDS, >= BWV + 4
    ld* h;         // LDS, >= BLZ + 1
    li* ired;      // LDS
    ld* part;      // LDS, PCG_PART
    V vp, vKp, vr, vz, td, zv, zv2;
    int n, m, r, d;
    int N2;
    double tau, beta;
    long long mv, lmv;  // FP64 and low-precision operator products
};
template <class V>
using LInst = __attribute__((address_space(3))) Inst<V>;

// ---- constraint operator --------------------------------------------------------
// The packed rows in FP64 (pairs) or their FP32 copy (quads), read as 16-byte pieces.
template <class T> struct Rows;
template <> struct Rows<double> {
    typedef double vec __attribute__((ext_vector_type(2)));
    static constexpr int W = 2;
    template <class B> static __device__ __forceinline__ const gd* base(const B& I) { return (const gd*)I.P; }
    template <class B> static __device__ __forceinline__ long pitch(const B& I) { return I.ldp; }
};
template <> struct Rows<float> {
    typedef float vec __attribute__((ext_vector_type(4)));
    static constexpr int W = 4;
    template <class B> static __device__ __forceinline__ const gf* base(const B& I) { return (const gf*)I.P32; }
    template <class B> static __device__ __forceinline__ long pitch(const B& I) { return I.ldp32; }
};
template <class T>
__device__ __forceinline__ typename Rows<T>::vec row_piece(const __attribute__((address_space(1))) T* row, int c) {
    typedef const __attribute__((address_space(1))) typename Rows<T>::vec gv;
    return ((gv*)row)[c];
}

// A value that every thread holds alike, as a scalar: arguments of a function
// that is not inlined arrive in vector registers.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// out[i] = alpha P_i . x + beta out[i] over the packed rows (x: ldr weights).
// A wave streams RW rows at once, its lanes over their pieces, PU pieces of
// each row in flight (16 loads per lane with four rows: 128 KB per workgroup,
// which is what one CU needs to draw on the last-level cache's bandwidth);
// the indices are clamped, so there is no serial tail.
template <class T, int RW, class O>
__device__ __forceinline__ void packed_rows_t(int m, int ldr, const __attribute__((address_space(1))) T* P,
                                              const gd* x, O out, double alpha, double beta) {
    typedef const __attribute__((address_space(1))) typename Rows<double>::vec gv2;
    constexpr int W = Rows<T>::W, PU = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hw = ldr / W;
    for (int i0 = wave * RW; i0 < m; i0 += BWV * RW) {
        double acc[RW];
        const __attribute__((address_space(1))) T* row[RW];
#pragma unroll
        for (int q = 0; q < RW; ++q) {
            acc[q] = 0.0;
            row[q] = P + (long)min(i0 + q, m - 1) * ldr;
        }
        for (int c0 = lane; c0 - lane < hw; c0 += 64 * PU) {
            typename Rows<T>::vec a[PU][RW];
            typename Rows<double>::vec xv[PU][W / 2];
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int cc = min(c0 + 64 * u, hw - 1);
#pragma unroll
                for (int q = 0; q < RW; ++q) a[u][q] = row_piece<T>(row[q], cc);
#pragma unroll
                for (int h = 0; h < W / 2; ++h) xv[u][h] = ((gv2*)x)[(W / 2) * cc + h];
            }
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const bool in = c0 + 64 * u < hw;
#pragma unroll
                for (int z = 0; z < W; ++z) {
                    const double xz = in ? xv[u][z / 2][z & 1] : 0.0;
#pragma unroll
                    for (int q = 0; q < RW; ++q) acc[q] += static_cast<double>(a[u][q][z]) * xz;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < RW; ++q) acc[q] = wave_sum_all(acc[q]);
        if (lane < RW && i0 + lane < m) {
            double v = acc[0];
#pragma unroll
            for (int q = 1; q < RW; ++q) v = lane == q ? acc[q] : v;
            out[i0 + lane] = (beta == 0.0) ? alpha * v : alpha * v + beta * out[i0 + lane];
        }
    }
    bsync();
}
template <class T, class O>
__device__ __noinline__ void wg_packed_rows(int m, int ldr, int rpw, const __attribute__((address_space(1))) T* P,
                                            const gd* x, O out, double alpha, double beta) {
    m = uni(m);
    ldr = uni(ldr);
    rpw = uni(rpw);
    if (rpw >= 4) packed_rows_t<T, 4>(m, ldr, P, x, out, alpha, beta);
    else if (rpw >= 2) packed_rows_t<T, 2>(m, ldr, P, x, out, alpha, beta);
    else packed_rows_t<T, 1>(m, ldr, P, x, out, alpha, beta);
}
// mw = packed weights of M: w_p (M_jk + M_kj) / 2, zero past N2
__device__ __noinline__ void wg_pack(int n, int N2, int ldr, const gi* pj, const gi* pk, const gd* M, gd* mw) {
    n = uni(n);
    for (int p = threadIdx.x; p < ldr; p += BT) {
        double v = 0.0;
        if (p < N2) {
            const int j = pj[p], k = pk[p];
            v = (j == k) ? M[j + j * n] : (M[j + k * n] + M[k + j * n]);
        }
        mw[p] = v;
    }
    bsync();
}
// out[i] = alpha <A_i, M> + beta out[i]
template <class T, class S, class O>
__device__ __forceinline__ void op_a(S s, const gd* M, O out, double alpha, double beta) {
    const int ldr = static_cast<int>(Rows<T>::pitch(s->I));
    wg_pack(s->n, s->N2, ldr, s->w.pj, s->w.pk, M, s->w.mw);
    wg_packed_rows<T, O>(s->m, ldr, s->I.rows_per_wave, Rows<T>::base(s->I), s->w.mw, out, alpha, beta);
}

// Y = A^T(u) as a full symmetric matrix: one thread per 16-byte piece of the
// packed columns, sixteen rows in flight (clamped, the factor zeroed past the
// end); where the pieces are fewer than the threads the rows are split over
// groups, added in order from LDS (part: 2 BT doubles).
template <class T, class U>
__device__ __noinline__ void wg_packed_cols(int n, int m, int N2, int ldr, const __attribute__((address_space(1))) T* P,
                                            U uv, ld* part, const gi* pj, const gi* pk, gd* Y) {
    n = uni(n);
    m = uni(m);
    N2 = uni(N2);
    ldr = uni(ldr);
    constexpr int W = Rows<T>::W, RU = 16;
    const int hw = ldr / W;
    auto span = [&](int c, int i0, int i1, double (&acc)[W]) {
#pragma unroll
        for (int q = 0; q < W; ++q) acc[q] = 0.0;
        for (int i = i0; i < i1; i += RU) {
            typename Rows<T>::vec a[RU];
#pragma unroll
            for (int q = 0; q < RU; ++q) a[q] = row_piece<T>(P + (long)min(i + q, m - 1) * ldr, c);
#pragma unroll
            for (int q = 0; q < RU; ++q) {
                const double v = uv[min(i + q, m - 1)], ui = i + q < i1 ? v : 0.0;
#pragma unroll
                for (int z = 0; z < W; ++z) acc[z] += static_cast<double>(a[q][z]) * ui;
            }
        }
    };
    auto put = [&](int p, double v) {
        if (p < N2) {
            const int j = pj[p], k = pk[p];
            Y[j + k * n] = v;
            Y[k + j * n] = v;
        }
    };
    const int groups = min(2 * BT / (hw * W), BT / hw);  // groups * hw * W sums fit part
    if (groups > 1) {
        const int g = threadIdx.x / hw, c = threadIdx.x % hw, per = (m + groups - 1) / groups;
        if (g < groups) {
            double acc[W];
            span(c, min(m, g * per), min(m, (g + 1) * per), acc);
#pragma unroll
            for (int q = 0; q < W; ++q) part[(g * hw + c) * W + q] = acc[q];
        }
        bsync();
        for (int p = threadIdx.x; p < N2; p += BT) {
            double v = 0.0;
            for (int g2 = 0; g2 < groups; ++g2) v += part[g2 * hw * W + p];
            put(p, v);
        }
    } else {
        for (int c = threadIdx.x; c < hw; c += BT) {
            double acc[W];
            span(c, 0, m, acc);
#pragma unroll
            for (int q = 0; q < W; ++q) put(W * c + q, acc[q]);
        }
    }
    bsync();
}
template <class T, class S, class U>
__device__ __forceinline__ void op_at(S s, U u, gd* Y) {
    wg_packed_cols<T, U>(s->n, s->m, s->N2, static_cast<int>(Rows<T>::pitch(s->I)), Rows<T>::base(s->I), u, s->part, s->w.pj,
                         s->w.pk, Y);
}

// ---- reformulation coordinates -------------------------------------------------------
__device__ void svec_ij(int c, int r, int& i, int& jj) {
    jj = 0;
    while (c >= r - jj) {
        c -= r - jj;
        ++jj;
    }
    i = jj + c;
}

// Hm (n x r) = [B; sqrt2 N] from v = [svec(B); vec(N)]
template <class S>
__device__ __forceinline__ void v_to_h(S s, const gd* v, gd* Hm) {
    const int n = s->n, r = s->r, nb = r * (r + 1) / 2;
    for (int t = threadIdx.x; t < n * r; t += BT) {
        const int a = t % n, b = t / n;
        double val;
        if (a < r) {
            const int i = a > b ? a : b, jj = a > b ? b : a;
            const int c = jj * r - jj * (jj - 1) / 2 + (i - jj);
            val = (i == jj) ? v[c] : v[c] * kIS2;
        } else {
            val = kS2 * v[nb + (a - r) + (n - r) * b];
        }
        Hm[t] = val;
    }
    bsync();
}

// out = [svec(sym F_top); sqrt2 vec(F_bot)]
template <class S>
__device__ __forceinline__ void f_to_v(S s, const gd* F, gd* out) {
    const int n = s->n, r = s->r, nb = r * (r + 1) / 2;
    for (int c = threadIdx.x; c < s->d; c += BT) {
        double val;
        if (c < nb) {
            int i, jj;
            svec_ij(c, r, i, jj);
            val = (i == jj) ? F[i + i * n] : kS2 * 0.5 * (F[i + jj * n] + F[jj + i * n]);
        } else {
            const int t = c - nb;
            const int k = t % (n - r), b = t / (n - r);
            val = kS2 * F[(r + k) + b * n];
        }
        out[c] = val;
    }
    bsync();
}

// M = (U Q^T + Q U^T) / 2, Q = first r columns of Gw
template <class S>
__device__ __forceinline__ void symlr(S s, const gd* U, gd* M) {
    const int n = s->n, r = s->r;
    for (int t = threadIdx.x; t < n * n; t += BT) {
        const int i = t % n, j = t / n;
        double a = 0.0;
        for (int b = 0; b < r; ++b) a += U[i + b * n] * s->w.Gw[j + b * n] + s->w.Gw[i + b * n] * U[j + b * n];
        M[t] = 0.5 * a;
    }
    bsync();
}

// ---- passes over the rows of script-A script-Q --------------------------------------
// The 16 lanes that share a row hold it in KC registers each (d <= 16 KC), so
// one pass gives the row's product AND the columns' sums with a factor known
// only after that product.  row(i, valid, av) is called for four rows per wave
// at a time, several such batches' loads in flight.
template <int KC, class S, class F>
__device__ __forceinline__ void aq_pass(S s, F&& row) {
    constexpr int PF = KC <= 4 ? 4 : (KC <= 8 ? 3 : 1);  // batches of rows in flight
    const int l = threadIdx.x & 15, slot = threadIdx.x >> 4, d = s->d, m = s->m;
    const int lda = static_cast<int>(s->w.ldaq);
    for (int i0 = slot; i0 - slot < m; i0 += PF * (BT / 16)) {
        double av[PF][KC];
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const gd* a = s->w.AQ + (long)min(i0 + q * (BT / 16), m - 1) * lda;
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const int c = l + 16 * k;
                const double v = a[min(c, d - 1)];
                av[q][k] = c < d ? v : 0.0;
            }
        }
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const int i = i0 + q * (BT / 16);
            if (i - slot < m) row(i, i < m, av[q]);
        }
    }
}
// the columns' sums of a pass into part[off + ...], one partial per wave
template <int KC, class S>
__device__ __forceinline__ void col_store(S s, int off, const double (&col)[KC]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const double v = rows4_sum(col[k]);
        if (lane < 16) s->part[off + wave * (16 * KC) + 16 * k + lane] = v;
    }
}
template <int KC, class S>
__device__ __forceinline__ double col_total(S s, int off, int c) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < BWV; ++q) v += s->part[off + q * (16 * KC) + c];
    return v;
}
// this lane's entries of a d-vector (zero past d)
template <int KC, class S, class X>
__device__ __forceinline__ void lane_vec(S s, X x, double (&xv)[KC]) {
    const int l = threadIdx.x & 15;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int c = l + 16 * k;
        const double v = x[min(c, s->d - 1)];
        xv[k] = c < s->d ? v : 0.0;
    }
}
template <int KC>
__device__ __forceinline__ double row_dot(const double (&a)[KC], const double (&x)[KC]) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < KC; ++k) t += a[k] * x[k];
    return row16_sum(t);
}

// vKp = K vp, the augmented operator (eq. augsys via the Section 5 products);
// returns vp . vKp.  lowp: its A E A^T block in low precision (the refinement
// sweeps' inner operator, as in the single-instance solver): A^T(u) and
// A(E Y E) over the FP32 rows, E Y E on the FP32 matrix cores.  The
// off-diagonal blocks are products with the explicit script-A script-Q that the
// preconditioner also uses, in FP64, and so is the bottom-right block.
// KC = 0: any d, the rows of AQ read twice.
template <int KC, class S>
__device__ __forceinline__ double op_k(S s, bool lowp) {
    const int n = s->n, m = s->m, d = s->d;
    auto& w = s->w;
    const double t2 = s->tau * s->tau;
    if (lowp) {
        op_at<float>(s, s->vp, w.Y);
        wg_sandwich<float>(n, w.E, w.Y, w.T1, w.Mm);
        op_a<float>(s, w.Mm, s->vKp, 1.0, 0.0);
        if (threadIdx.x == 0) s->lmv += 1;
    } else {
        op_at<double>(s, s->vp, w.Y);
        wg_sandwich<double>(n, w.E, w.Y, w.T1, w.Mm);
        op_a<double>(s, w.Mm, s->vKp, 1.0, 0.0);
        if (threadIdx.x == 0) s->mv += 1;
    }
    double pk = 0.0;
    const int l = threadIdx.x & 15;
    if constexpr (KC > 0) {
        double v[KC], col[KC];
        lane_vec<KC>(s, s->vp + m, v);
#pragma unroll
        for (int k = 0; k < KC; ++k) col[k] = 0.0;
        aq_pass<KC>(s, [&](int i, bool ok, const double (&av)[KC]) {
            const int ic = min(i, m - 1);
            const double u = ok ? s->vp[ic] : 0.0;
            const double o = s->vKp[ic] + row_dot<KC>(av, v);
            if (ok && l == 0) {
                s->vKp[i] = o;
                pk += u * o;
            }
#pragma unroll
            for (int k = 0; k < KC; ++k) col[k] += u * av[k];
        });
        col_store<KC>(s, 0, col);
        bsync();
        for (int c = threadIdx.x; c < d; c += BT) {
            const double vc = s->vp[m + c], o = col_total<KC>(s, 0, c) - t2 * w.sig[c] * vc;
            s->vKp[m + c] = o;
            pk += vc * o;
        }
    } else {
        wg_rows(m, d, w.AQ, static_cast<int>(w.ldaq), s->vp + m, [&](int i, double t) {
            if (l == 0) {
                const double o = s->vKp[i] + t;
                s->vKp[i] = o;
                pk += s->vp[i] * o;
            }
        });
        wg_cols(m, d, w.AQ, static_cast<int>(w.ldaq), s->vp, s->part, [&](int c, double t) {
            const double vc = s->vp[m + c], o = t - t2 * w.sig[c] * vc;
            s->vKp[m + c] = o;
            pk += vc * o;
        });
    }
    return wg_sum(pk, s->red);
}

// z = P^{-1} [r; 0] (Section 6: block elimination with P = [beta I, AQ; AQ^T,
// -tau^2 Sigma], then one step of iterative refinement, as in the
// single-instance solver) for the residual r in vr, whose products (AQ)^T r
// the caller has left in td, scaled by -1 / beta; returns r . z.  vKp is
// overwritten (with the refinement residual's top block).
template <int KC, class S>
__device__ __forceinline__ double precond(S s) {
    const int m = s->m, d = s->d, ldc = s->bp.dmax, lda = static_cast<int>(s->w.ldaq);
    auto& w = s->w;
    const double ib = 1.0 / s->beta, beta = s->beta, t2 = s->tau * s->tau;
    const int l = threadIdx.x & 15;
    wg_rows(d, d, w.Cm, ldc, s->td, [&](int c, double t) {
        if (l == 0) s->zv[c] = -t;
    });
    bsync();
    // z1 = (r - AQ zv) / beta, rho = r - AQ zv - beta z1, and both products with (AQ)^T
    if constexpr (KC > 0) {
        double x[KC], c1[KC], c2[KC];
        lane_vec<KC>(s, s->zv, x);
#pragma unroll
        for (int k = 0; k < KC; ++k) c1[k] = c2[k] = 0.0;
        aq_pass<KC>(s, [&](int i, bool ok, const double (&av)[KC]) {
            const double f = s->vr[min(i, m - 1)], t = row_dot<KC>(av, x);
            const double z = ok ? ib * (f - t) : 0.0, rho = ok ? f - t - beta * z : 0.0;
            if (ok && l == 0) {
                s->vz[i] = z;
                s->vKp[i] = rho;
            }
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                c1[k] += z * av[k];
                c2[k] += rho * av[k];
            }
        });
        col_store<KC>(s, 0, c1);
        col_store<KC>(s, BWV * 16 * KC, c2);
        bsync();
        for (int c = threadIdx.x; c < d; c += BT)
            s->td[c] = t2 * w.sig[c] * s->zv[c] - col_total<KC>(s, 0, c) - ib * col_total<KC>(s, BWV * 16 * KC, c);
        bsync();
    } else {
        wg_rows(m, d, w.AQ, lda, s->zv, [&](int i, double t) {
            if (l == 0) {
                const double f = s->vr[i], z = ib * (f - t);
                s->vz[i] = z;
                s->vKp[i] = f - t - beta * z;
            }
        });
        bsync();
        wg_cols(m, d, w.AQ, lda, s->vz, s->part, [&](int c, double t) { s->td[c] = t2 * w.sig[c] * s->zv[c] - t; });
        wg_cols(m, d, w.AQ, lda, s->vKp, s->part, [&](int c, double t) { s->td[c] -= ib * t; });
    }
    wg_rows(d, d, w.Cm, ldc, s->td, [&](int c, double t) {
        if (l == 0) s->zv2[c] = -t;
    });
    bsync();
    double rz = 0.0;
    if constexpr (KC > 0) {
        double x[KC];
        lane_vec<KC>(s, s->zv2, x);
        aq_pass<KC>(s, [&](int i, bool ok, const double (&av)[KC]) {
            const int ic = min(i, m - 1);
            const double t = row_dot<KC>(av, x);
            const double z = s->vz[ic] + ib * (s->vKp[ic] - t);
            if (ok && l == 0) {
                s->vz[i] = z;
                rz += s->vr[i] * z;
            }
        });
    } else {
        wg_rows(m, d, w.AQ, lda, s->zv2, [&](int i, double t) {
            if (l == 0) {
                const double z = s->vz[i] + ib * (s->vKp[i] - t);
                s->vz[i] = z;
                rz += s->vr[i] * z;
            }
        });
    }
    for (int c = threadIdx.x; c < d; c += BT) s->vz[m + c] = s->zv[c] + s->zv2[c];
    return wg_sum(rz, s->red);
}

// dy = u / tau^2, dX = E (A^T u - tau^2 C~) E + sym(U Q^T)  (eq. recover)
template <class S>
__device__ __noinline__ void recover(S s, const gd* x, const gd* Ct, gd* dX, gd* dy) {
    const int n = s->n, m = s->m, r = s->r;
    auto& w = s->w;
    const double t2 = s->tau * s->tau;
    for (int i = threadIdx.x; i < m; i += BT) dy[i] = x[i] / t2;
    bsync();
    op_at<double>(s, x, w.Y);
    wg_axpby(n * n, -t2, Ct, 1.0, w.Y, w.Y);
    wg_gemm(false, false, n, n, n, 1.0, w.Y, n, w.E, n, 0.0, w.T1, n);
    v_to_h(s, x + m, w.Hm);
    wg_gemm(false, false, n, r, n, 1.0, w.Gw, n, w.Hm, n, 0.0, w.U, n);
    symlr(s, w.U, dX);
    wg_gemm(false, false, n, n, n, 1.0, w.E, n, w.T1, n, 1.0, dX, n);
    wg_symmetrize(n, dX);
}

// Indefinite PCG (Definition pcg, Corollary pcg) on K x = g from the x
// given, with the FP64 operator or its low-precision form: stops when
// ||r_u|| <= tol_rel ||r_u(0)||; returns the iteration count, negative
// (-its - 1) when maxit was reached first.  ref and rr receive ||r_u(0)|| and
// the final ||r_u||.  The bottom block of the residual is zero throughout.
//
// An iteration is a chain of phases of one workgroup, each bound by the
// latency of its loads, sums and barrier, so they are merged: the update of x
// and r, the new norm and (AQ)^T r share a pass over AQ, and so do the row
// product and the two column products of the preconditioner's refinement.
template <int KC, class S>
__device__ __noinline__ int pcg_t(S s, bool lowp, const gd* g, gd* x, double tol_rel, int maxit, double& ref,
                                     double& rr) {
    const int m = s->m, d = s->d, N = m + d;
    auto& w = s->w;
    const double ib = 1.0 / s->beta;
    const int l = threadIdx.x & 15;
    wg_copy(N, x, s->vp);
    for (int c = threadIdx.x; c < d; c += BT) s->vr[m + c] = 0.0;
    double rz = 1.0, tol = 0.0;
    int it = 0;
    bool conv = false, first = true;
    while (true) {
        const double pkp = op_k<KC>(s, lowp);
        // the first product is K x: r = g - K x; afterwards x += alpha p, r -= alpha K p
        const double alpha = rz / pkp;
        auto update = [&](int i) {
            double ri;
            if (first) {
                ri = g[i] - s->vKp[i];
            } else {
                ri = s->vr[i] - alpha * s->vKp[i];
                if (l == 0) x[i] += alpha * s->vp[i];
            }
            if (l == 0) s->vr[i] = ri;
            return ri;
        };
        double rs = 0.0;
        if (!first)
            for (int c = threadIdx.x; c < d; c += BT) x[m + c] += alpha * s->vp[m + c];
        if constexpr (KC > 0) {
            double col[KC];
#pragma unroll
            for (int k = 0; k < KC; ++k) col[k] = 0.0;
            aq_pass<KC>(s, [&](int i, bool ok, const double (&av)[KC]) {
                const double ri = ok ? update(i) : 0.0;
                if (l == 0) rs += ri * ri;
#pragma unroll
                for (int k = 0; k < KC; ++k) col[k] += ri * av[k];
            });
            col_store<KC>(s, 0, col);
            rr = sqrt(wg_sum(rs, s->red));
            for (int c = threadIdx.x; c < d; c += BT) s->td[c] = -ib * col_total<KC>(s, 0, c);
            bsync();
        } else {
            for (int i0 = threadIdx.x >> 4; i0 < m; i0 += BT / 16) {
                const double ri = update(i0);
                if (l == 0) rs += ri * ri;
            }
            rr = sqrt(wg_sum(rs, s->red));
            wg_cols(m, d, w.AQ, static_cast<int>(w.ldaq), s->vr, s->part, [&](int c, double t) { s->td[c] = -ib * t; });
        }
        if (first) {
            ref = rr;
            tol = tol_rel * (ref > 0.0 ? ref : 1.0);
        } else {
            ++it;
        }
        if (!(rr > tol)) {
            conv = isfinite(rr);
            break;
        }
        if (it >= maxit) break;
        const double rzn = precond<KC>(s);
        const double bk = first ? 0.0 : rzn / rz;
        rz = rzn;
        for (int t = threadIdx.x; t < N; t += BT) s->vp[t] = first ? s->vz[t] : s->vz[t] + bk * s->vp[t];
        bsync();
        first = false;
    }
    return conv ? it : -it - 1;
}
template <class S>
__device__ __forceinline__ int pcg(S s, bool lowp, const gd* g, gd* x, double tol_rel, int maxit, double& ref,
                                   double& rr) {
    if (s->d <= 64) return pcg_t<4>(s, lowp, g, x, tol_rel, maxit, ref, rr);
    if (s->d <= 128) return pcg_t<8>(s, lowp, g, x, tol_rel, maxit, ref, rr);
    if (s->d <= 16 * PCG_KC) return pcg_t<PCG_KC>(s, lowp, g, x, tol_rel, maxit, ref, rr);
    return pcg_t<0>(s, lowp, g, x, tol_rel, maxit, ref, rr);
}

// vKp = K vp in FP64 for the refinement sweeps
template <class S>
__device__ __noinline__ void residual_product(S s) {
    op_k<0>(s, false);
}

// The Newton system of eq. Newt-eps by eq. augsys started at [0; -Sigma^{-1}
// Q^T c], then eq. recover; returns the Krylov iteration count (negative when
// the tolerance was not met).  With the low-precision operator: FP64
// refinement sweeps, each a low-precision PCG run on the FP64 residual g - K x
// (bottom block zero) from zero to refine_tol, or to the reduction still
// missing to inner_tol when that is larger.
template <class S>
__device__ __noinline__ int inner_solve(S s, const gd* bt, const gd* Ct, gd* dX, gd* dy) {
    const int n = s->n, m = s->m, r = s->r, d = s->d, N = m + d;
    auto& w = s->w;
    const double t2 = s->tau * s->tau;
    // g = [b~ + tau^2 A(E C~ E); tau^2 Q^T c]
    wg_gemm(false, false, n, n, n, 1.0, Ct, n, w.E, n, 0.0, w.T1, n);
    wg_gemm(false, false, n, n, n, 1.0, w.E, n, w.T1, n, 0.0, w.Mm, n);
    op_a<double>(s, w.Mm, w.vg, t2, 0.0);
    wg_axpby(m, 1.0, bt, 1.0, w.vg, w.vg);
    wg_gemm(false, false, n, r, n, 1.0, Ct, n, w.Gw, n, 0.0, w.YQ, n);
    wg_gemm(true, false, n, r, n, 1.0, w.Gw, n, w.YQ, n, 0.0, w.F, n);
    f_to_v(s, w.F, w.vtmp);
    for (int c = threadIdx.x; c < d; c += BT) {
        w.vg[m + c] = t2 * w.vtmp[c];
        w.vx[m + c] = -w.vtmp[c] / w.sig[c];
    }
    for (int i = threadIdx.x; i < m; i += BT) w.vx[i] = 0.0;
    bsync();
    const double tol = s->bp.inner_tol;
    const bool lowp = s->bp.lowp != 0;
    int its = 0;
    bool conv = false;
    double ref = 0.0;
    for (int sweep = 0;; ++sweep) {
        const gd* rhs = w.vg;
        gd* sol = w.vx;
        double ptol = tol;
        if (lowp) {
            wg_copy(N, w.vx, s->vp);
            residual_product(s);
            for (int t = threadIdx.x; t < N; t += BT) w.vres[t] = (t < m) ? w.vg[t] - s->vKp[t] : 0.0;
            bsync();
            const double rr = sqrt(wg_dot(m, w.vres, w.vres, s->red));
            if (sweep == 0) ref = rr;
            if (!(rr > tol * (ref > 0.0 ? ref : 1.0))) {
                conv = isfinite(rr);
                break;
            }
            if (!isfinite(rr) || sweep >= s->bp.max_refine || its >= s->bp.inner_maxit) break;
            wg_fill(N, w.vdx, 0.0);
            ptol = fmax(s->bp.refine_tol, 0.5 * tol * ref / (rr > 0.0 ? rr : 1.0));
            rhs = w.vres;
            sol = w.vdx;
        }
        double r0, r1;
        const int it = pcg(s, lowp, rhs, sol, ptol, s->bp.inner_maxit - its, r0, r1);
        its += it >= 0 ? it : -it - 1;
        if (!lowp) {
            conv = it >= 0;
            break;
        }
        if (!isfinite(r1)) break;
        wg_axpby(N, 1.0, w.vdx, 1.0, w.vx, w.vx);
    }
    recover(s, w.vx, Ct, dX, dy);
    return conv ? its : -its - 1;
}

// Largest alpha with L L^T + alpha D PSD, from lambda_min(L^{-1} D L^{-T}).
template <class S>
__device__ __noinline__ double max_step(S s, const gd* Li, const gd* D) {
    const int n = s->n;
    auto& w = s->w;
    wg_gemm(false, false, n, n, n, 1.0, Li, n, D, n, 0.0, w.T1, n);
    wg_gemm(false, true, n, n, n, 1.0, w.T1, n, Li, n, 0.0, w.Tp, n);
    const double lmin = wg_lanczos_min(n, w.Tp, w.Q, w.td, w.ab, s->red, s->h, s->ired);
    return lmin >= 0.0 ? 1e300 : -1.0 / lmin;
}

// Shrink alpha by 0.9 until M + alpha D has a Cholesky factor; negative on failure.
template <class S>
__device__ __noinline__ double guard_step(S s, const gd* M, const gd* D, double alpha) {
    const int n = s->n;
    for (int t = 0; t < 40; ++t) {
        wg_axpby(n * n, 1.0, M, alpha, D, s->w.T1);
        if (wg_potrf(n, s->w.T1, n) == 0) return alpha;
        alpha *= 0.9;
    }
    return -1.0;
}

struct BResid {
    double mu, pobj, dobj, relgap, pinf, dinf;
};

template <class S>
__device__ __noinline__ void residuals(S s, BResid& R) {
    const int n = s->n, m = s->m;
    const int nn = n * n;
    auto& w = s->w;
    op_a<double>(s, w.X, w.rp, -1.0, 0.0);
    wg_axpby(m, 1.0, (const gd*)s->I.b, 1.0, w.rp, w.rp);
    op_at<double>(s, w.y, w.Y);
    for (int t = threadIdx.x; t < nn; t += BT) w.Rd[t] = ((const gd*)s->I.C)[t] - w.Y[t] - w.S[t];
    bsync();
    wg_symmetrize(n, w.Rd);
    R.mu = wg_dot(nn, w.X, w.S, s->red) / n;
    R.pobj = wg_dot(nn, (const gd*)s->I.C, w.X, s->red);
    R.dobj = wg_dot(m, (const gd*)s->I.b, w.y, s->red);
    R.relgap = fabs(R.pobj - R.dobj) / (1.0 + fabs(R.pobj) + fabs(R.dobj));
    R.pinf = sqrt(wg_dot(m, w.rp, w.rp, s->red)) / (1.0 + s->I.bnorm);
    R.dinf = sqrt(wg_dot(nn, w.Rd, w.Rd, s->red)) / (1.0 + s->I.Cnorm);
}

// Scaling point, eigen-split, E, Sigma, script-A script-Q and C^{-1}.
// Returns 0, or a negative status.
template <class S>
__device__ __noinline__ int scaling(S s) {
    const int n = s->n, m = s->m;
    const int nn = n * n;
    auto& w = s->w;
    wg_copy(nn, w.X, w.L);
    if (wg_potrf(n, w.L, n)) return kENumeric;
    wg_copy(nn, w.S, w.R);
    if (wg_potrf(n, w.R, n)) return kENumeric;
    wg_trtri(n, w.L, w.Linv);
    wg_trtri(n, w.R, w.Rinv);
    const double tol = fmax(n, 16) * 1.1102230246251565e-16;
    // NT factor: R^T L = U D V^T, G = L V D^{-1/2}, G^{-1} = D^{1/2} V^T L^{-1}
    wg_gemm(true, false, n, n, n, 1.0, w.R, n, w.L, n, 0.0, w.T1, n);
    wg_identity(n, w.Vs, 1.0);
    if (wg_jacobi(n, w.T1, w.Vs, w.dnt, w.T2, w.nrm, w.rank, tol, 60, s->red) >= 60) return kENumeric;
    wg_gemm(false, false, n, n, n, 1.0, w.L, n, w.Vs, n, 0.0, w.T1, n);
    wg_scale_cols(n, n, w.T1, w.dnt, -0.5, w.G);
    wg_gemm(true, false, n, n, n, 1.0, w.Vs, n, w.Linv, n, 0.0, w.T1, n);
    wg_scale_rows(n, w.T1, w.dnt, 0.5, w.Ginv);
    // eigen-decomposition of W = G G^T: one-sided Jacobi on G^T
    wg_transpose(n, w.G, w.Gt);
    wg_identity(n, w.Gw, 1.0);
    if (wg_jacobi(n, w.Gt, w.Gw, w.lam, w.T2, w.nrm, w.rank, tol, 60, s->red) >= 60) return kENumeric;
    for (int k = threadIdx.x; k < n; k += BT) w.lam[k] = w.lam[k] * w.lam[k];
    bsync();
    // rank rule, tau, d (Experiments section; eq. EQSigdef)
    const int rhat = min(s->I.rmax, n - 1);
    int r = 1;
    double bv = -1.0;
    for (int i = 1; i <= rhat; ++i) {
        const double v = w.lam[i - 1] / w.lam[i];
        if (v > bv) {
            bv = v;
            r = i;
        }
    }
    const double tau = 0.5 * w.lam[r];
    const int sd = n * r - r * (r - 1) / 2;
    // beta = median(eig E)^2 * mean ||A_i||_F^2
    for (int k = threadIdx.x; k < n; k += BT) w.evE[k] = (k < r) ? 1.0 : w.lam[k] / tau;
    bsync();
    for (int k = threadIdx.x; k < n; k += BT) {
        int rk = 0;
        for (int j = 0; j < n; ++j) rk += (w.evE[j] < w.evE[k]) || (w.evE[j] == w.evE[k] && j < k);
        w.srt[rk] = w.evE[k];
    }
    bsync();
    const double med = (n & 1) ? w.srt[n / 2] : 0.5 * (w.srt[n / 2 - 1] + w.srt[n / 2]);
    const double beta = med * med * s->I.mean_a2;
    if (threadIdx.x == 0) {
        s->r = r;
        s->tau = tau;
        s->d = sd;
        s->beta = beta;
    }
    bsync();
    // E = G_w diag(e) G_w^T and Sigma
    wg_scale_cols(n, n, w.Gw, w.evE, 1.0, w.T1);
    wg_gemm(false, true, n, n, n, 1.0, w.T1, n, w.Gw, n, 0.0, w.E, n);
    wg_symmetrize(n, w.E);
    {
        const int nb = r * (r + 1) / 2;
        for (int c = threadIdx.x; c < sd; c += BT) {
            double v;
            if (c < nb) {
                int i, jj;
                svec_ij(c, r, i, jj);
                v = 1.0 / (w.lam[i] * w.lam[jj] - tau * tau);
            } else {
                const int t = c - nb;
                const int k = t % (n - r), b = t / (n - r);
                v = 1.0 / ((w.lam[b] - tau) * w.lam[r + k]);
            }
            w.sig[c] = v;
        }
        bsync();
    }
    // script-A script-Q: row i from F_i = G_w^T A_i Q, constraints in groups
    const int grp = s->I.aq_group;
    const int nb = r * (r + 1) / 2;
    for (int i0 = 0; i0 < m; i0 += grp) {
        const int gc = min(grp, m - i0);
        // T_g = A_i Q (n x r) for the group, A_i read from its packed row
        for (int t = threadIdx.x; t < gc * n * r; t += BT) {
            const int g = t / (n * r);
            const int rem = t % (n * r);
            const int j = rem % n, b = rem / n;
            const gd* Pi = (const gd*)s->I.P + (long)(i0 + g) * s->I.ldp;
            double a = 0.0;
#pragma unroll 8
            for (int k = 0; k < n; ++k) {
                const int hi = j > k ? j : k, lo = j > k ? k : j;
                const int p = lo * n - lo * (lo - 1) / 2 + (hi - lo);
                a += Pi[p] * w.Gw[k + (long)b * n];
            }
            w.Taq[t] = a;
        }
        bsync();
        // F_i = G_w^T T_i, written straight into row i of AQ
        for (int t = threadIdx.x; t < gc * sd; t += BT) {
            const int g = t / sd, c = t % sd;
            const gd* Ti = w.Taq + (long)g * n * r;
            auto Fab = [&](int a, int b) {
                double v = 0.0;
#pragma unroll 8
                for (int j = 0; j < n; ++j) v += w.Gw[j + a * n] * Ti[j + b * n];
                return v;
            };
            double val;
            if (c < nb) {
                int a, b;
                svec_ij(c, r, a, b);
                val = (a == b) ? Fab(a, a) : kS2 * 0.5 * (Fab(a, b) + Fab(b, a));
            } else {
                const int t2 = c - nb;
                const int k = t2 % (n - r), b = t2 / (n - r);
                val = kS2 * Fab(r + k, b);
            }
            w.AQ[(long)(i0 + g) * w.ldaq + c] = val;
        }
        bsync();
    }
    // C = tau^2 Sigma + (AQ)^T (AQ) / beta (AQ row-major = column-major d x m), then C^{-1}
    wg_gemm(false, true, sd, sd, m, 1.0 / beta, w.AQ, w.ldaq, w.AQ, w.ldaq, 0.0, w.Cm, s->bp.dmax);
    for (int c = threadIdx.x; c < sd; c += BT) w.Cm[c + (long)c * s->bp.dmax] += tau * tau * w.sig[c];
    bsync();
    if (wg_spd_inverse(sd, w.Cm, s->bp.dmax, w.colk)) return kENumeric;
    return 0;
}

// The interior-point method of solver.hip for one instance.
template <class S>
__device__ __forceinline__ void solve_one(S s, const BInst* inst, BOut* out) {
    if (threadIdx.x == 0) {
        const BInst I = *inst;
        *(BInst*)&s->I = I;
        s->n = I.n;
        s->m = I.m;
        s->r = 1;
        s->d = 1;
        s->N2 = static_cast<int>(I.N2);
        s->mv = 0;
        s->lmv = 0;
        wg_tile = I.gemm_tile;
    }
    bsync();
    auto& w = s->w;
    auto& I = s->I;
    auto& bp = s->bp;
    ld* red = s->red;
    const int n = s->n, m = s->m;
    const int nn = n * n;
    for (int t = threadIdx.x; t < nn; t += BT) {
        const int j = t % n, k = t / n;
        if (j >= k) {
            const int p = k * n - k * (k - 1) / 2 + (j - k);
            w.pj[p] = j;
            w.pk[p] = k;
        }
    }
    wg_identity(n, w.X, I.xi);
    wg_identity(n, w.S, I.eta);
    wg_fill(m + 8, w.y, 0.0);
    BOut o{};
    o.status = kEStall;
    long long pcg = 0;
    int its = 0;
    BResid R{};
    for (int k = 0; k <= bp.max_ipm_iter; ++k) {
        residuals(s, R);
        if (R.relgap <= bp.gap_tol && R.pinf <= bp.feas_tol && R.dinf <= bp.feas_tol) {
            o.status = 0;
            break;
        }
        if (k == bp.max_ipm_iter) break;
        int rc = scaling(s);
        if (rc) {
            o.status = rc;
            break;
        }
        // the predictor (b~ = r_p, C~ = R_d + S), then the corrector, through one
        // inlined copy of the Newton system's solve
        wg_axpby(nn, 1.0, w.Rd, 1.0, w.S, w.Ct);
        bool solved = true;
        for (int ph = 0; ph < 2; ++ph) {
            gd* DX = ph == 0 ? w.dXa : w.dX;
            gd* DS = ph == 0 ? w.dSa : w.dS;
            gd* Dy = ph == 0 ? w.dya : w.dy;
            const int pi = inner_solve(s, w.rp, w.Ct, DX, Dy);
            if (pi < 0) {
                solved = false;
                break;
            }
            pcg += pi;
            op_at<double>(s, Dy, w.Y);
            wg_axpby(nn, 1.0, w.Rd, -1.0, w.Y, DS);
            if (ph == 1) break;
            const double ap = fmin(1.0, max_step(s, w.Linv, w.dXa));
            const double ad = fmin(1.0, max_step(s, w.Rinv, w.dSa));
            const double xds = wg_dot(nn, w.X, w.dSa, red), dxs = wg_dot(nn, w.dXa, w.S, red);
            const double dxds = wg_dot(nn, w.dXa, w.dSa, red);
            const double mu_aff = (R.mu * n + ad * xds + ap * dxs + ap * ad * dxds) / n;
            double sg = fmin(1.0, fmax(0.0, mu_aff / R.mu));
            sg = sg * sg * sg;
            // corrector: H from Dx = G^{-1} dXa G^{-T}, Ds = G^T dSa G; C~ = R_d - G^{-T} H G^{-1}
            wg_gemm(false, false, n, n, n, 1.0, w.Ginv, n, w.dXa, n, 0.0, w.T1, n);
            wg_gemm(false, true, n, n, n, 1.0, w.T1, n, w.Ginv, n, 0.0, w.Tp, n);   // Dx
            wg_gemm(true, false, n, n, n, 1.0, w.G, n, w.dSa, n, 0.0, w.T1, n);
            wg_gemm(false, false, n, n, n, 1.0, w.T1, n, w.G, n, 0.0, w.Hc, n);     // Ds
            wg_gemm(false, false, n, n, n, 1.0, w.Tp, n, w.Hc, n, 0.0, w.T2, n);    // Dx Ds
            for (int t = threadIdx.x; t < nn; t += BT) {
                const int i = t % n, j = t / n;
                double v = -(w.T2[i + j * n] + w.T2[j + i * n]);
                if (i == j) v += 2.0 * (sg * R.mu - w.dnt[i] * w.dnt[i]);
                w.Hc[t] = v / (w.dnt[i] + w.dnt[j]);
            }
            bsync();
            wg_gemm(true, false, n, n, n, 1.0, w.Ginv, n, w.Hc, n, 0.0, w.T1, n);
            wg_gemm(false, false, n, n, n, 1.0, w.T1, n, w.Ginv, n, 0.0, w.T2, n);
            wg_axpby(nn, 1.0, w.Rd, -1.0, w.T2, w.Ct);
            wg_symmetrize(n, w.Ct);
        }
        if (!solved) {
            o.status = kENotConv;
            break;
        }
        const double frac = bp.step_frac;
        const double apc = guard_step(s, w.X, w.dX, fmin(1.0, frac * max_step(s, w.Linv, w.dX)));
        const double adc = guard_step(s, w.S, w.dS, fmin(1.0, frac * max_step(s, w.Rinv, w.dS)));
        if (apc < 0.0 || adc < 0.0) {
            o.status = kENumeric;
            break;
        }
        wg_axpby(nn, apc, w.dX, 1.0, w.X, w.X);
        wg_axpby(m, adc, w.dy, 1.0, w.y, w.y);
        wg_axpby(nn, adc, w.dS, 1.0, w.S, w.S);
        wg_symmetrize(n, w.X);
        wg_symmetrize(n, w.S);
        ++its;
    }
    if (o.status != 0) residuals(s, R);
    if (threadIdx.x == 0) {
        o.iterations = its;
        o.pcg = pcg;
        o.matvecs = s->mv;
        o.lp_matvecs = s->lmv;
        o.pobj = R.pobj;
        o.dobj = R.dobj;
        o.relgap = R.relgap;
        o.pinf = R.pinf;
        o.dinf = R.dinf;
        o.mu = R.mu;
        *out = o;
    }
    if (I.Xout) wg_copy(nn, w.X, (gd*)I.Xout);
    if (I.yout) wg_copy(m, w.y, (gd*)I.yout);
    bsync();
}

// VL: the Krylov vectors in LDS (after the partial sums), else in the
// workgroup's scratch.
template <bool VL>
__global__ __launch_bounds__(BT) void batched_kernel(const BInst* __restrict__ insts, const int* __restrict__ order,
                                                     int count, BParams bp, double* __restrict__ scratch,
                                                     int* __restrict__ queue, BOut* __restrict__ outs) {
    typedef std::conditional_t<VL, ld*, gd*> V;
    __shared__ double red[BWV + 4];
    __shared__ double h[BLZ + 1];
    __shared__ int ired[2];
    __shared__ Inst<V> inst;
    extern __shared__ double dyn[];  // PCG_PART, then the vectors
    LInst<V>* s = (LInst<V>*)&inst;
    if (threadIdx.x == 0) {
        const Work w = carve((gd*)scratch + (long)blockIdx.x * bp.per_wg, bp);
        inst.w = w;
        inst.bp = bp;
        s->red = (ld*)red;
        s->h = (ld*)h;
        s->ired = (li*)ired;
        s->part = (ld*)dyn;
        if constexpr (VL) {
            const int NV = bp.mmax + bp.dmax + 8;
            ld* v = (ld*)dyn + PCG_PART;
            s->vp = v;
            s->vKp = v + NV;
            s->vr = v + 2 * NV;
            s->vz = v + 3 * NV;
            s->td = v + 4 * NV;
            s->zv = v + 4 * NV + bp.dmax;
            s->zv2 = v + 4 * NV + 2 * bp.dmax;
        } else {
            s->vp = w.vp;
            s->vKp = w.vKp;
            s->vr = w.vr;
            s->vz = w.vz;
            s->td = w.td;
            s->zv = w.td2;
            s->zv2 = w.td3;
        }
    }
    while (true) {
        if (threadIdx.x == 0) ired[1] = atomicAdd(queue, 1);
        bsync();
        const int q = ired[1];
        bsync();
        if (q >= count) break;  // every workgroup ends here once the queue is empty
        const int i = order[q];
        solve_one(s, insts + i, outs + i);
    }
}

}  // namespace

// ---- host side ------------------------------------------------------------------------
namespace {

struct Staged {
    std::vector<BInst> insts;
    DevBuf<double> data;  // packed rows, b and C of every instance
    DevBuf<float> data32; // FP32 copies of the packed rows (low-precision inner solves)
    BParams bp{};
};

constexpr int STAGE_THREADS = 8;

long dim_d(int n, int r) { return (long)n * r - (long)r * (r - 1) / 2; }

void stage(const sdp_problem* probs, int count, const sdp_options& o, hipStream_t st, const BatchTune* tune,
           Staged& S) {
    require(count >= 1, "count must be positive");
    S.insts.resize(count);
    long total = 0;
    int nmax = 2, mmax = 1, rcap = 1;
    long N2max = 1;
    for (int i = 0; i < count; ++i) {
        const sdp_problem& p = probs[i];
        require(p.a_kind == SDP_A_DENSE, "the batched solver takes dense constraint matrices");
        require(p.n >= 2 && p.m >= 1 && p.A && p.b && p.C, "bad batched problem");
        require(!p.on_device, "batched problems are read from host memory");
        const long N2 = (long)p.n * (p.n + 1) / 2;
        require(p.m <= N2, "m exceeds n(n+1)/2");
        const long ldp = round_up(N2, 2);
        total += (long)p.m * ldp + round_up(p.m, 2) + round_up((long)p.n * p.n, 2);
        nmax = std::max(nmax, p.n);
        mmax = std::max(mmax, p.m);
        N2max = std::max(N2max, ldp);
        rcap = std::max(rcap, std::min(std::max(1, o.rank_max), p.n - 1));
    }
    S.data.alloc(total);
    // low-precision inner solves: every instance's rows again in FP32, rows of
    // ldp32 = round_up(N2, 4) floats so that they load as 16-byte quads
    const bool lowp = o.inner_prec == SDP_PREC_F32;
    long total32 = 0;
    if (lowp) {
        for (int i = 0; i < count; ++i) {
            const long N2 = (long)probs[i].n * (probs[i].n + 1) / 2;
            total32 += (long)probs[i].m * round_up(N2, 4);
        }
        S.data32.alloc(total32);
    }
    // where each instance's block goes; every block an even number of doubles,
    // so that the packed rows stay 16-byte aligned
    std::vector<long> off(count + 1, 0), off32(count + 1, 0);
    for (int i = 0; i < count; ++i) {
        const sdp_problem& p = probs[i];
        const long N2 = (long)p.n * (p.n + 1) / 2;
        off[i + 1] = off[i] + (long)p.m * round_up(N2, 2) + round_up(p.m, 2) + round_up((long)p.n * p.n, 2);
        off32[i + 1] = off32[i] + (lowp ? (long)p.m * round_up(N2, 4) : 0);
    }
    auto pack = [&](int i, double* host, float* host32) {
        const sdp_problem& p = probs[i];
        const int n = p.n, m = p.m;
        const long nn = (long)n * n;
        const long N2 = (long)n * (n + 1) / 2;
        const long ldp = round_up(N2, 2);
        double a2 = 0.0, amax = 0.0, ratio = 0.0, bn = 0.0, cn = 0.0;
        for (int r = 0; r < m; ++r) {
            const double* Ar = p.A + (long)r * nn;
            double nr2 = 0.0;
            long q = 0;
            for (int k = 0; k < n; ++k)
                for (int j = k; j < n; ++j, ++q) {
                    const double v = 0.5 * (Ar[j + (long)k * n] + Ar[k + (long)j * n]);
                    require(std::isfinite(v), "A has a non-finite entry");
                    host[(long)r * ldp + q] = v;
                    nr2 += (j == k ? 1.0 : 2.0) * v * v;
                }
            a2 += nr2;
            amax = std::max(amax, std::sqrt(nr2));
            ratio = std::max(ratio, (1.0 + std::fabs(p.b[r])) / (1.0 + std::sqrt(nr2)));
            bn += p.b[r] * p.b[r];
            host[(long)m * ldp + r] = p.b[r];
        }
        for (long t = 0; t < nn; ++t) {
            const int j = static_cast<int>(t % n), k = static_cast<int>(t / n);
            const double v = 0.5 * (p.C[t] + p.C[k + (long)j * n]);
            host[(long)m * ldp + round_up(m, 2) + t] = v;
            cn += v * v;
        }
        const long ldp32 = round_up(N2, 4);
        if (lowp)
            for (int r = 0; r < m; ++r)
                for (long q = 0; q < N2; ++q) host32[(long)r * ldp32 + q] = static_cast<float>(host[(long)r * ldp + q]);
        BInst& I = S.insts[i];
        I.n = n;
        I.m = m;
        I.rmax = std::max(1, std::min(o.rank_max, n - 1));
        const BatchForm form = batch_form(n);  // without a tuning
        I.rows_per_wave = tune ? tune[i].rows_per_wave : form.rows_per_wave;
        I.aq_group = tune ? tune[i].aq_group : 8;
        I.gemm_tile = tune ? (tune[i].gemm_tile ? tune[i].gemm_tile : 32) : form.gemm_tile;
        require(I.rows_per_wave >= 1 && I.rows_per_wave <= 4 && I.aq_group >= 1 && I.aq_group <= 16 &&
                    (I.gemm_tile == 16 || I.gemm_tile == 32),
                "batch tune out of range (rows_per_wave 1..4, aq_group 1..16, gemm_tile 0, 16 or 32)");
        I.N2 = N2;
        I.ldp = ldp;
        I.ldp32 = ldp32;
        I.P32 = lowp ? S.data32.get() + off32[i] : nullptr;
        I.P = S.data.get() + off[i];
        I.b = S.data.get() + off[i] + (long)m * ldp;
        I.C = S.data.get() + off[i] + (long)m * ldp + round_up(m, 2);
        I.mean_a2 = a2 / m;
        I.bnorm = std::sqrt(bn);
        I.Cnorm = std::sqrt(cn);
        I.xi = std::max({10.0, std::sqrt((double)n), n * ratio});
        I.eta = std::max({10.0, std::sqrt((double)n), 1.0 + std::max(amax, I.Cnorm)});
        I.Xout = nullptr;
        I.yout = nullptr;
    };
    // Groups of instances up to STAGE_BYTES are packed by several threads into
    // one host buffer and copied at once: packing one by one on one thread, with
    // a copy and a synchronisation each, took 66 ms for 256 instances of n = 16 ..
    // 24; this takes 23.  An error is that of the first instance that has one, as
    // in a plain loop.
    constexpr long STAGE_BYTES = 64L << 20;
    std::vector<double> host;
    std::vector<float> host32;
    for (int i0 = 0, i1; i0 < count; i0 = i1) {
        for (i1 = i0 + 1; i1 < count && 8 * (off[i1 + 1] - off[i0]) <= STAGE_BYTES; ++i1) {}
        host.assign(off[i1] - off[i0], 0.0);
        host32.assign(off32[i1] - off32[i0], 0.0f);
        std::atomic<int> next{i0};
        std::vector<std::exception_ptr> errs(i1 - i0);
        auto work = [&] {
            for (int i = next++; i < i1; i = next++) {
                try {
                    pack(i, host.data() + (off[i] - off[i0]), host32.data() + (off32[i] - off32[i0]));
                } catch (...) {
                    errs[i - i0] = std::current_exception();
                }
            }
        };
        // a thread pays from a megabyte on; without one, this thread does the work
        const long mb = 8 * (off[i1] - off[i0]) >> 20;
        const int nt = static_cast<int>(std::min<long>({STAGE_THREADS - 1, mb, i1 - i0 - 1}));
        run_shared(nt, work);
        for (auto& e : errs)
            if (e) std::rethrow_exception(e);
        WC_HIP(hipMemcpyAsync(S.data.get() + off[i0], host.data(), sizeof(double) * host.size(), hipMemcpyHostToDevice,
                              st));
        if (lowp)
            WC_HIP(hipMemcpyAsync(S.data32.get() + off32[i0], host32.data(), sizeof(float) * host32.size(),
                                  hipMemcpyHostToDevice, st));
        WC_HIP(hipStreamSynchronize(st));
    }
    BParams& bp = S.bp;
    bp.nmax = nmax;
    bp.mmax = mmax;
    bp.rcap = rcap;
    bp.dmax = static_cast<int>(round_up(dim_d(nmax, rcap) + 1, 8));
    bp.N2max = N2max;
    const long nn = (long)nmax * nmax;
    const long NV = mmax + bp.dmax + 8;
    auto r8 = [](long c) { return (c + 7) & ~7L; };
    bp.per_wg = 24 * r8(nn) + r8((long)nmax * (BLZ + 1)) + 5 * r8(mmax + 8) + 5 * r8(nmax) + r8(2L * nmax) +
                r8(bp.dmax) + 4 * r8((long)nmax * rcap) + 11 * r8(NV) + 3 * r8(bp.dmax) +
                r8((long)mmax * bp.dmax) + r8((long)bp.dmax * bp.dmax) + r8(bp.dmax) + 2 * r8(N2max + 8) +
                r8(16L * nmax * rcap) + r8(2L * BLZ) + 2 * r8(N2max / 2 + 8) + r8(nmax / 2 + 8);
    bp.inner_tol = o.inner_tol;
    bp.inner_maxit = o.inner_maxit;
    bp.gap_tol = o.gap_tol;
    bp.feas_tol = o.feas_tol;
    bp.max_ipm_iter = o.max_ipm_iter;
    bp.step_frac = o.step_frac;
    bp.lowp = lowp ? 1 : 0;
    bp.max_refine = o.max_refine;
    bp.refine_tol = o.refine_tol > 0 ? o.refine_tol : 1e-6;
}

// Launch the persistent kernel over `sel` (indices into S.insts) and wait.
double run(Staged& S, const std::vector<int>& sel, hipStream_t st, std::vector<BOut>& outs) {
    const int count = static_cast<int>(sel.size());
    // largest instances first
    std::vector<int> order(sel);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        const BInst &x = S.insts[a], &y = S.insts[b];
        return (double)x.m * x.N2 > (double)y.m * y.N2;
    });
    int dev = 0, cus = 0;
    WC_HIP(hipGetDevice(&dev));
    WC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int grid = std::max(1, std::min(count, 2 * cus));
    DevBuf<BInst> dinst(S.insts.size());
    DevBuf<int> dorder(count), queue(1);
    DevBuf<BOut> douts(S.insts.size());
    DevBuf<double> scratch((size_t)grid * S.bp.per_wg);
    WC_HIP(hipMemcpyAsync(dinst.get(), S.insts.data(), sizeof(BInst) * S.insts.size(), hipMemcpyHostToDevice, st));
    WC_HIP(hipMemcpyAsync(dorder.get(), order.data(), sizeof(int) * count, hipMemcpyHostToDevice, st));
    WC_HIP(hipMemsetAsync(queue.get(), 0, sizeof(int), st));
    WC_HIP(hipMemsetAsync(douts.get(), 0, sizeof(BOut) * S.insts.size(), st));
    WC_HIP(hipStreamSynchronize(st));
    const auto t0 = std::chrono::steady_clock::now();
    // the Krylov vectors in LDS where they fit beside the partial sums (n = 128
    // at rank_max 10 takes 140 KB); a larger instance keeps them in its scratch
    int lds_max = 0;
    WC_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    const size_t part_b = sizeof(double) * PCG_PART;
    const size_t vec_b = sizeof(double) * (4 * ((size_t)S.bp.mmax + S.bp.dmax + 8) + 3 * (size_t)S.bp.dmax);
    if (part_b + vec_b + 2048 <= static_cast<size_t>(lds_max))
        hipLaunchKernelGGL(batched_kernel<true>, dim3(grid), dim3(BT), part_b + vec_b, st, dinst.get(), dorder.get(),
                           count, S.bp, scratch.get(), queue.get(), douts.get());
    else
        hipLaunchKernelGGL(batched_kernel<false>, dim3(grid), dim3(BT), part_b, st, dinst.get(), dorder.get(), count,
                           S.bp, scratch.get(), queue.get(), douts.get());
    WC_LAUNCH_CHECK();
    WC_HIP(hipStreamSynchronize(st));
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    outs.resize(S.insts.size());
    WC_HIP(hipMemcpy(outs.data(), douts.get(), sizeof(BOut) * S.insts.size(), hipMemcpyDeviceToHost));
    return ms;
}

}  // namespace

void solve_batched(const sdp_problem* probs, int count, const sdp_options* opt, hipStream_t st, sdp_result* results,
                   double* const* X_out, double* const* y_out, const BatchTune* tune) {
    sdp_options o;
    if (opt) o = *opt;
    else sdp_default_options(&o);
    Staged S;
    stage(probs, count, o, st, tune, S);
    for (int i = 0; i < count; ++i) {
        S.insts[i].Xout = X_out ? X_out[i] : nullptr;
        S.insts[i].yout = y_out ? y_out[i] : nullptr;
    }
    std::vector<int> sel(count);
    std::iota(sel.begin(), sel.end(), 0);
    std::vector<BOut> outs;
    const double ms = run(S, sel, st, outs);
    for (int i = 0; i < count; ++i) {
        sdp_result& r = results[i];
        const BOut& b = outs[i];
        r.status = b.status;
        r.iterations = b.iterations;
        r.pcg_iterations = b.pcg;
        r.newton_matvecs = b.matvecs;
        r.pobj = b.pobj;
        r.dobj = b.dobj;
        r.relgap = b.relgap;
        r.pinf = b.pinf;
        r.dinf = b.dinf;
        r.mu = b.mu;
        r.time_ms = ms;
        r.lp_matvecs = b.lp_matvecs;
    }
}

void autotune_batched(const sdp_problem* probs, int count, const sdp_options* opt, hipStream_t st, BatchTune* out,
                      double* bucket_ms) {
    sdp_options o;
    if (opt) o = *opt;
    else sdp_default_options(&o);
    o.max_ipm_iter = 2;  // time the first iterations only
    // pass settings x the wave tile of the workgroup's MFMA products; 16 x 16
    // wave tiles are the faster ones up to n = 32 (batch_form), so they are tried
    // in the first bucket only
    const BatchTune cands[] = {{1, 4, 32}, {2, 8, 32}, {4, 8, 32}, {4, 16, 32},
                               {1, 4, 16}, {2, 8, 16}, {4, 8, 16}, {4, 16, 16}};
    const int ncand_all = sizeof(cands) / sizeof(cands[0]);
    auto bucket = [](int n) { return n < 48 ? 0 : (n < 96 ? 1 : 2); };
    for (int i = 0; i < count; ++i) out[i] = cands[1];
    for (int bk = 0; bk < 3; ++bk) {
        std::vector<int> idx;
        for (int i = 0; i < count && (int)idx.size() < 8; ++i)
            if (bucket(probs[i].n) == bk) idx.push_back(i);
        if (bucket_ms) bucket_ms[bk] = 0.0;
        if (idx.empty()) continue;
        std::vector<sdp_problem> sample;
        for (int i : idx) sample.push_back(probs[i]);
        int best = 1;
        double best_ms = 1e300;
        const int ncand = bk == 0 ? ncand_all : 4;
        for (int c = 0; c < ncand; ++c) {
            std::vector<BatchTune> tt(sample.size(), cands[c]);
            Staged S;
            stage(sample.data(), (int)sample.size(), o, st, tt.data(), S);
            std::vector<int> sel(sample.size());
            std::iota(sel.begin(), sel.end(), 0);
            std::vector<BOut> outs;
            const double ms = run(S, sel, st, outs);
            if (ms < best_ms) {
                best_ms = ms;
                best = c;
            }
        }
        if (bucket_ms) bucket_ms[bk] = best_ms;
        for (int i = 0; i < count; ++i)
            if (bucket(probs[i].n) == bk) out[i] = cands[best];
    }
}

}  // namespace wc
