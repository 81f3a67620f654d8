// The augmented operator's kernels for dense constraint rows beyond the shared
// building blocks: the middle of the product for small n and the last pass.
#pragma once

#include "common.hpp"

namespace wc {

// Largest n for which dense_mid runs: past it one workgroup takes longer than the
// launches it saves.  newton_apply in us, with it and with the products split over
// the chip: n = 16 13 and 24, n = 40 23 and 32, n = 64 32 and 37 (m = 1664 37 and 41), n =
// 65 39 and 38 (m = 1716 47 and 41), n = 80 46 and 43.
constexpr int DENSE_MID_N = 64;

// mw = packed weights of E Y E (zero past N2, ldp entries), with Y = A^T(u) given
// as the nparts slab partial sums of its packed entries (row pitch pstride): the
// sums, both products and the packing in one workgroup.  n <= DENSE_MID_N.
void dense_mid(hipStream_t st, int n, long N2, long ldp, int nparts, const double* part, long pstride, const int* pj,
               const int* pk, const double* E, double* mw);

// mw = packed weights of sum_s P_s over `splits` n x n partial products (ld n).
void reduce_pack(hipStream_t st, int n, long N2, long ldp, int splits, const double* P, const int* pj, const int* pk,
                 double* mw);

// The last pass of the operator, in one launch:
//   out[i]     = P_i . mw + AQ_i . v            (i < m, the packed rows P and AQ row-major)
//   out[m + c] = AQt_c . u - t2 sig_c v_c       (c < d, AQt = AQ^T row-major)
// P and mw in FP64, or in FP32 with FP64 accumulation.  AQ and AQt rows are
// 16-byte aligned; u and v need no more than their own alignment.  t0 / t1 as
// for packed_rows.
template <class T>
void op_rows(hipStream_t st, int m, long k, const T* P, long ldp, const T* mw, int d, const double* AQ, long ldaq,
             const double* AQt, long ldaqt, const double* u, const double* v, const double* sig, double t2,
             double* out, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr);

// The preconditioner's passes over AQ (m x d, row-major) and AQt = AQ^T for the
// block elimination with P = [beta I, AQ; AQ^T, -tau^2 Sigma] and its refinement
// step, each with the vector work around it (ib = 1 / beta).  Rows 16-byte
// aligned and zero padded; f, z1, rho and zv aligned likewise.
//   precond_down:  td = h - ib AQt f
//   precond_up:    t = AQ zv;  z1 = ib (f - t);  rho = (f - t) - beta z1
//   precond_down2: td = (h - AQt z1 + t2 sig zv) - ib AQt rho
//   precond_up2:   z1 += ib (rho - AQ zv2);  zout = zv + zv2
void precond_down(hipStream_t st, int m, int d, const double* AQt, long ldaqt, const double* f, const double* h,
                  double ib, double* td);
void precond_up(hipStream_t st, int m, int d, const double* AQ, long ldaq, const double* zv, const double* f, double ib,
                double beta, double* z1, double* rho);
void precond_down2(hipStream_t st, int m, int d, const double* AQt, long ldaqt, const double* z1, const double* rho,
                   const double* h, const double* sig, double t2, const double* zv, double ib, double* td);
void precond_up2(hipStream_t st, int m, int d, const double* AQ, long ldaq, const double* zv, const double* zv2,
                 const double* rho, double ib, double* z1, double* zout);

}  // namespace wc
