// Blocked Cholesky factorisation and triangular inversion (FP64, gfx950).
//
// potrf: 32-column panels, left-looking inside 256-column outer panels: one
// launch updates a panel, factors its diagonal block and solves the rows below;
// the trailing matrix takes an MFMA GEMM per outer panel.
// trtri: the 32 x 32 diagonal blocks, then diagonal blocks up to 1024 by column
// blocks in one launch, then recursive 2 x 2 blocking, inv([L11 0; L21 L22]) =
// [L11^{-1} 0; -L22^{-1} L21 L11^{-1} L22^{-1}].
#include "common.hpp"

namespace wc {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int PNB = 32;

// The value of lane `l` (the same in all lanes), as a scalar.
__device__ __forceinline__ double lane_value(double v, int l) {
    const long long x = __double_as_longlong(v);
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), l));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x >> 32), l));
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<long long>(lo));
}

// a[q - 1] = a[q] - x c[q] for q in [Q0, W): c in LDS, read by all lanes at
// once.  (The entries as scalars by v_readlane cost 45 cycles each here, two
// readlanes and a wait per product; from LDS 15.)
template <int Q0, int W>
__device__ __forceinline__ void shift_update(double (&a)[32], double x, const double* c) {
    double l[32];
#pragma unroll
    for (int q = Q0; q < W; ++q) l[q] = c[q];
#pragma unroll
    for (int q = Q0; q < W; ++q) a[q - 1] = fma(-x, l[q], a[q]);
}

// 1 / sqrt(d) and sqrt(d) from the hardware estimate: two Newton steps and a
// correction of the root.  A pivot that is not positive counts as 1.
struct Pivot {
    double rs, sd;
};
__device__ __forceinline__ Pivot take_pivot(double d, int j, int nb, int offset, int& bad) {
    const bool ok = d > 0.0;
    bad = (!ok && bad == 0 && j < nb) ? offset + j + 1 : bad;
    d = ok ? d : 1.0;
    double rs = __builtin_amdgcn_rsq(d);
    const double h = -0.5 * d;
    rs = rs * fma(h * rs, rs, 1.5);
    rs = rs * fma(h * rs, rs, 1.5);
    const double s0 = d * rs;
    const double sd = fma(0.5 * rs, fma(-s0, s0, d), s0);
    const bool inf = d == __builtin_inf();  // as a root and a division would leave it
    return Pivot{inf ? 0.0 : rs, inf ? d : sd};
}

// Two matrices of one size may be factored or inverted by one launch
// (blockIdx.y): X and S of a scaling point.
struct Pair {
    double* p[2];
};

constexpr int LT = 2 * PNB + 1;
// One wave factors the panel in T (T[c]: column c; the block's 32 rows, then 32
// rows below it): a row per lane in registers, column by column.
__device__ __forceinline__ void panel_columns(int nb, int offset, int* info, double (*T)[LT]) {
    const int lane = threadIdx.x & 63;
    double a[PNB];
#pragma unroll
    for (int c = 0; c < PNB; ++c) a[c] = T[c][lane];
#pragma unroll
    for (int c = 0; c < PNB; ++c)  // the identity past the block's end
        if (lane < PNB && (lane >= nb || c > lane)) a[c] = lane == c ? 1.0 : 0.0;
    int bad = 0;
    Pivot pv = take_pivot(lane_value(a[0], 0), 0, nb, offset, bad);
    auto columns = [&](auto width, int j0) {
        constexpr int W = decltype(width)::value;  // entries left of a row at column j0
        const int j1 = min(j0 + 8, nb);
#pragma unroll 1
        for (int j = j0; j < j1; ++j) {
            const double a0 = a[0] * pv.rs;
            T[j][lane] = lane == j ? pv.sd : a0;  // one wave: its LDS accesses are in order
            a[0] = fma(-a0, lane_value(a0, j + 1), a[1]);
            pv = take_pivot(lane_value(a[0], j + 1), j + 1, nb, offset, bad);
            shift_update<2, W>(a, a0, &T[j][j]);
        }
    };
    columns(std::integral_constant<int, 32>{}, 0);
    columns(std::integral_constant<int, 24>{}, 8);
    columns(std::integral_constant<int, 16>{}, 16);
    columns(std::integral_constant<int, 8>{}, 24);
    if (info != nullptr && lane == 0 && bad && *info == 0) *info = bad;
}

// Panel k of the outer panel that starts at k0: its 32 columns (nb < 32 only at
// the end of the matrix) take the updates of columns k0 .. k - 1, the diagonal
// block is factored and the rows below it are solved against it, in one launch
// (an update GEMM, an LDS factorisation of the block and a solve took 10 + 21 +
// 10 us at n = 300; this takes 15).
// A workgroup owns 32 rows below the block and works the block out itself.  The
// update is seven 16 x 16 MFMA tiles, a quarter of K per wave (four operand loads
// for seven products; tiles split over the waves load four times as much).
// Then one wave holds a row per lane, the block's in lanes 0 .. 31: a column's
// entries L[k][j] go through LDS to all lanes and update every row at once,
// without a barrier.  The row shifts down one entry per column (the
// FMA's destination), so one short loop serves 8 columns: unrolled over 32
// the code is 25 KB, and it took 27 us.  Bound by the chain of 32 columns (380
// cycles each at 8 entries left, 860 at 32).
// The other workgroups read the block while workgroup 0 ends, so the factor is
// not written over it but, when rest > 0, into the strict upper triangle
// (transposed; its diagonal into the column after the block), which
// potrf_finish_kernel puts in place.
__global__ __launch_bounds__(256) void potrf_panel_kernel(int n, int k0, int k, int nb, Pair mats, long lda,
                                                          int* __restrict__ info) {
    __shared__ double T[PNB][LT];  // T[c]: column c of the block's rows, then of the 32 rows
    double* A = mats.p[blockIdx.y];
    double* Akk = A + k + (long)k * lda;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rest = n - k - nb, r0 = blockIdx.x * PNB;
    // row i of T, clamped to one that is there
    auto row_of = [&](int i) { return i < PNB ? min(i, nb - 1) : (rest > 0 ? nb + min(r0 + i - PNB, rest - 1) : 0); };
    // 8 of the 32 columns per wave; the block's upper triangle is not read
    double base[8];
    {
        const int i = row_of(lane);
#pragma unroll
        for (int q = 0; q < 8; ++q) base[q] = Akk[i + (long)min(min(wave * 8 + q, nb - 1), i) * lda];
    }
    // a quarter of K per wave: the block's three lower tiles and the rows' four,
    // from two operands of each kind
    d4 acc[7];
#pragma unroll
    for (int t = 0; t < 7; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    const int K = k - k0;
    if (K > 0) {
        constexpr int U = 4;
        const int ks = wave * (K / 4);  // K is a multiple of 32
        const double* Lk = A + k + (long)(k0 + ks + (lane >> 4)) * lda;
        const double* f[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) f[t] = Lk + row_of(16 * t + (lane & 15));
        double c[4][U], d[4][U];
        auto load = [&](double (&v)[4][U], int kk) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // past the wave's share: its last entries once more, not used
                const long o = (long)min(kk + 4 * u, K / 4 - 4) * lda;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t][u] = f[t][o];
            }
        };
        auto mul = [&](const double (&v)[4][U], int kk) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kk + 4 * u >= K / 4) break;
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0][u], v[0][u], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1][u], v[0][u], acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1][u], v[1][u], acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[2][u], v[0][u], acc[3], 0, 0, 0);
                acc[4] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[2][u], v[1][u], acc[4], 0, 0, 0);
                acc[5] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[3][u], v[0][u], acc[5], 0, 0, 0);
                acc[6] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[3][u], v[1][u], acc[6], 0, 0, 0);
            }
        };
        load(c, 0);
        load(d, 4 * U);
#pragma unroll 1
        for (int kk = 0; kk < K / 4; kk += 8 * U) {
            mul(c, kk);
            load(c, kk + 8 * U);
            mul(d, kk + 4 * U);
            load(d, kk + 12 * U);
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) T[wave * 8 + q][lane] = base[q];
    __syncthreads();
    if (K > 0) {
        for (int w = 0; w < 4; ++w) {  // in wave order
            if (wave == w) {
#pragma unroll
                for (int t = 0; t < 7; ++t) {
                    const int ti = t == 0 ? 0 : t < 3 ? 1 : t < 5 ? 2 : 3, tj = t < 3 ? (t == 2) : (t == 4 || t == 6);
#pragma unroll
                    for (int v = 0; v < 4; ++v) T[16 * tj + (lane & 15)][16 * ti + (lane >> 4) + 4 * v] -= acc[t][v];
                }
            }
            __syncthreads();
        }
    }
    if (wave == 0) panel_columns(nb, k, blockIdx.x == 0 ? info + blockIdx.y : nullptr, T);
    __syncthreads();
    // workgroup 0 writes the factor: transposed, its diagonal past the block, or in place
    const bool mine = lane >= PNB && r0 + lane - PNB < rest, own = blockIdx.x == 0 && lane < nb;
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
        const int c = wave * 8 + q;
        if (c >= nb) break;
        const double v = T[c][lane];
        if (mine) Akk[nb + r0 + lane - PNB + (long)c * lda] = v;
        if (own && rest == 0 && lane >= c) Akk[lane + (long)c * lda] = v;
        if (own && rest > 0 && lane == c) Akk[lane + (long)nb * lda] = v;
        if (rest > 0 && blockIdx.x == 0 && lane < c) Akk[lane + (long)c * lda] = T[lane][c];
    }
}

// The diagonal blocks' factors from the upper triangle into place, and the
// strict upper triangle cleared.  Blocks start at the multiples of PNB; the
// last one is already in place.
__global__ __launch_bounds__(256) void potrf_finish_kernel(int n, Pair mats, long lda) {
    double* A = mats.p[blockIdx.y];
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)n * n) return;
    const int i = static_cast<int>(t % n), j = static_cast<int>(t / n);
    const int b = i / PNB, e = b * PNB + PNB;  // the block of row i ends before e
    if (i == j) {
        if (e < n) {
            A[i + (long)i * lda] = A[i + (long)e * lda];
            A[i + (long)e * lda] = 0.0;
        }
    } else if (i < j) {
        if (j / PNB == b && e < n) A[j + (long)i * lda] = A[i + (long)j * lda];
        if (j != e) A[i + (long)j * lda] = 0.0;
    }
}

__global__ void zero_info(int* p) { p[threadIdx.x] = 0; }

// A panel's update reads only its outer panel (PNB_OUTER columns, or all of a
// matrix up to twice that); the rest of the trailing matrix takes one GEMM of
// rank PNB_OUTER per outer panel, so it is streamed n / PNB_OUTER times.
constexpr int PNB_OUTER = 256;
static void potrf_pair(hipStream_t st, int n, Pair m, int count, long lda, int* info) {
    hipLaunchKernelGGL(zero_info, dim3(1), dim3(count), 0, st, info);
    WC_LAUNCH_CHECK();
    if (n <= 0) return;
    const int outer = n > 2 * PNB_OUTER ? PNB_OUTER : n;
    for (int k0 = 0; k0 < n; k0 += outer) {
        const int kend = std::min(n, k0 + outer);  // columns [k0, kend) form the outer panel
        for (int k = k0; k < kend; k += PNB) {
            const int kb = std::min(PNB, kend - k);
            hipLaunchKernelGGL(potrf_panel_kernel, dim3(std::max(1, cdiv(n - k - kb, PNB)), count), dim3(256), 0, st, n,
                               k0, k, kb, m, lda, info);
            WC_LAUNCH_CHECK();
        }
        const int rest = n - kend;
        for (int q = 0; q < count && rest > 0; ++q) {
            // the trailing matrix past the outer panel, in one update of rank kend - k0
            const double* Pb = m.p[q] + kend + (long)k0 * lda;
            double* A22 = m.p[q] + kend + (long)kend * lda;
            dgemm(st, false, true, rest, rest, kend - k0, -1.0, Pb, lda, Pb, lda, 1.0, A22, lda, /*lower_only=*/true);
        }
    }
    hipLaunchKernelGGL(potrf_finish_kernel, dim3(cdiv((long)n * n, 256), count), dim3(256), 0, st, n, m, lda);
    WC_LAUNCH_CHECK();
}
void potrf(hipStream_t st, int n, double* A, long lda, int* info) { potrf_pair(st, n, Pair{{A, A}}, 1, lda, info); }
void potrf2(hipStream_t st, int n, double* A, double* B, long lda, int* info) {
    potrf_pair(st, n, Pair{{A, B}}, 2, lda, info);
}

struct ConstPair {
    const double* p[2];
};

// Workgroup b inverts the diagonal block [PNB b, min(PNB b + PNB, n)) by one
// wave: lane j holds column j of the inverse, which shifts as above.
__global__ __launch_bounds__(64) void trtri_leaf_kernel(int n, ConstPair Ls, long ldl, Pair Xs, long ldx) {
    const int b0 = blockIdx.x * PNB, nb = min(PNB, n - b0);
    const double* L = Ls.p[blockIdx.y] + b0 + (long)b0 * ldl;
    double* X = Xs.p[blockIdx.y] + b0 + (long)b0 * ldx;
    const int lane = threadIdx.x, li = min(lane, nb - 1);
    __shared__ double Lc[PNB][2 * PNB];  // Lc[c]: column c of the block (the second half is not used)
    __shared__ double rd[PNB];
    const double* Lr = L + li;
    double x[PNB];
#pragma unroll
    for (int c = 0; c < PNB; ++c) x[c] = Lr[(long)min(c, li) * ldl];
    const double r = 1.0 / Lr[(long)li * ldl];
#pragma unroll
    for (int c = 0; c < PNB; ++c) {
        Lc[c][lane] = x[c];
        x[c] = lane == c ? 1.0 : 0.0;
    }
    if (lane < PNB) rd[lane] = r;
    __syncthreads();
    auto columns = [&](auto width, int j0) {
        constexpr int W = decltype(width)::value;
        const int j1 = min(j0 + 8, nb);
#pragma unroll 1
        for (int j = j0; j < j1; ++j) {
            const double x0 = x[0] * rd[j];
            if (lane < nb) X[j + (long)lane * ldx] = x0;  // zero above the diagonal
            shift_update<1, W>(x, x0, &Lc[j][j]);
        }
    };
    columns(std::integral_constant<int, 32>{}, 0);
    columns(std::integral_constant<int, 24>{}, 8);
    columns(std::integral_constant<int, 16>{}, 16);
    columns(std::integral_constant<int, 8>{}, 24);
}

// The rest of the inverse of the TR_MAX x TR_MAX diagonal blocks: a workgroup
// owns 16 columns of X, which it keeps in LDS, and walks down the 32-row blocks,
//   X_I = -L_II^{-1} sum_{K < I} L_IK X_K,
// the sum split over its four waves (MFMA).  All columns at once in one launch,
// where the two products per level of a recursion were 2 (n / 32 - 1) launches
// of 8 to 11 us (n = 300: 150 us to 20).  Bound by the chain of blocks, a
// round of loads and two barriers each.
constexpr int TR_MAX = 1024;  // TR_MAX x 16 doubles of LDS
constexpr int TR_C = 16;
__global__ __launch_bounds__(256) void trtri_cols_kernel(int n, ConstPair Ls, long ldl, Pair Xs, long ldx) {
    extern __shared__ double Xc[];              // Xc[(row - c0's block) * 16 + column]
    __shared__ double red[4][2][16 * TR_C];
    const double* L = Ls.p[blockIdx.y];
    double* X = Xs.p[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.x * TR_C, lo = c0 / PNB * PNB;
    const int end = min(n, c0 / TR_MAX * TR_MAX + TR_MAX);
    const int nc = min(TR_C, n - c0);
    // zeros above the column block's first diagonal block
    for (int j = wave; j < nc; j += 4)
        for (int i = lane; i < lo; i += 64) X[i + (long)(c0 + j) * ldx] = 0.0;
    for (int t = tid; t < PNB * TR_C; t += 256) {
        const int i = t % PNB, j = t / PNB;
        Xc[i * TR_C + j] = (lo + i < n && j < nc) ? X[lo + i + (long)(c0 + j) * ldx] : 0.0;
    }
    __syncthreads();
    const int l15 = lane & 15, l4 = lane >> 4;
    for (int I = lo + PNB; I < end; I += PNB) {
        // L_II^{-1} for the second product, in flight through the first
        double f[8];
        const int row2 = min(I + 16 * (wave & 1) + l15, n - 1);
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = X[row2 + (long)min(I + l4 + 4 * u, n - 1) * ldx];
        const int kw = (I - lo) / 4;  // this wave's share of K, a multiple of 8
        const int ks = wave * kw;
        const double* p0 = L + min(I + l15, n - 1) + (long)(lo + ks + l4) * ldl;
        const double* p1 = L + min(I + 16 + l15, n - 1) + (long)(lo + ks + l4) * ldl;
        const double* xb = Xc + (ks + l4) * TR_C + l15;
        d4 s0{0.0, 0.0, 0.0, 0.0}, s1{0.0, 0.0, 0.0, 0.0};
        constexpr int U = 8;
        int kk = 0;
#pragma unroll 1
        for (; kk + 4 * U <= kw; kk += 4 * U) {
            double a0[U], a1[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a0[u] = p0[(long)(kk + 4 * u) * ldl];
                a1[u] = p1[(long)(kk + 4 * u) * ldl];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double x = xb[(kk + 4 * u) * TR_C];
                s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[u], x, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[u], x, s1, 0, 0, 0);
            }
        }
#pragma unroll 1
        for (; kk < kw; kk += 8) {
            double a0[2], a1[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                a0[u] = p0[(long)(kk + 4 * u) * ldl];
                a1[u] = p1[(long)(kk + 4 * u) * ldl];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double x = xb[(kk + 4 * u) * TR_C];
                s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[u], x, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[u], x, s1, 0, 0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            red[wave][0][(l4 + 4 * v) * TR_C + l15] = s0[v];
            red[wave][1][(l4 + 4 * v) * TR_C + l15] = s1[v];
        }
        __syncthreads();
        if (wave < 2) {
            d4 x{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (wave == 0 && u >= 4) break;  // the inverse's upper triangle
                const int o = ((l4 + 4 * u) & 15) * TR_C + l15, t = u >> 2;
                const double s = (red[0][t][o] + red[1][t][o]) + (red[2][t][o] + red[3][t][o]);
                // a ragged last block has no columns past n
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(f[u], I + l4 + 4 * u < n ? s : 0.0, x, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * wave + l4 + 4 * v;
                Xc[(I - lo + i) * TR_C + l15] = -x[v];
                if (I + i < n && l15 < nc) X[I + i + (long)(c0 + l15) * ldx] = -x[v];
            }
        }
        __syncthreads();
    }
}

// Every split is at a multiple of TR_MAX from the start of the matrix, so the
// leaves (n <= TR_MAX) are the aligned diagonal blocks, already inverted.
static void trtri_rec(hipStream_t st, int n, const double* L, long ldl, double* X, long ldx, double* work) {
    if (n <= TR_MAX) return;
    int n1 = static_cast<int>(round_up(n / 2, TR_MAX));
    if (n1 >= n) n1 = n - TR_MAX;
    int n2 = n - n1;
    trtri_rec(st, n1, L, ldl, X, ldx, work);
    trtri_rec(st, n2, L + n1 + (long)n1 * ldl, ldl, X + n1 + (long)n1 * ldx, ldx, work);
    // T = L21 X11 (n2 x n1), stored in work with leading dimension n2
    dgemm(st, false, false, n2, n1, n1, 1.0, L + n1, ldl, X, ldx, 0.0, work, n2);
    // X21 = -X22 T
    dgemm(st, false, false, n2, n1, n2, -1.0, X + n1 + (long)n1 * ldx, ldx, work, n2, 0.0, X + n1, ldx);
}

static void trtri_pair(hipStream_t st, int n, ConstPair L, long ldl, Pair X, long ldx, int count, double* work) {
    if (n <= 0) return;
    hipLaunchKernelGGL(trtri_leaf_kernel, dim3(cdiv(n, PNB), count), dim3(64), 0, st, n, L, ldl, X, ldx);
    WC_LAUNCH_CHECK();
    const size_t lds = sizeof(double) * TR_C * round_up(std::min(n, TR_MAX), PNB);
    hipLaunchKernelGGL(trtri_cols_kernel, dim3(cdiv(n, TR_C), count), dim3(256), lds, st, n, L, ldl, X, ldx);
    WC_LAUNCH_CHECK();
    for (int q = 0; q < count; ++q) trtri_rec(st, n, L.p[q], ldl, X.p[q], ldx, work);
}
void trtri(hipStream_t st, int n, const double* L, long ldl, double* Linv, long ldi, double* work) {
    trtri_pair(st, n, ConstPair{{L, L}}, ldl, Pair{{Linv, Linv}}, ldi, 1, work);
}
void trtri2(hipStream_t st, int n, const double* L, const double* M, long ld, double* Linv, double* Minv,
            double* work) {
    trtri_pair(st, n, ConstPair{{L, M}}, ld, Pair{{Linv, Minv}}, ld, 2, work);
}

}  // namespace wc
