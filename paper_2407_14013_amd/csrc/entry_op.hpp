// Products with script-A script-Q for entry sampling without forming it
// (Section 6), with the vector work around them.
#pragma once

#include <functional>

#include "common.hpp"

namespace wc {

// The LP columns of script-A script-Q (t of them, 0 without an LP block): T, B by
// columns and by rows, each coordinate's position in T (-1 when out).
struct EntryLp {
    int t;
    const int *Tl, *cptr, *crow, *rptr, *rcol, *pos;
    const double *cval, *rval;
};

// The constraint pattern and the scaling's vectors: pairs jk, symmetric CSR
// pattern (row j lists each pair (j, p) or (p, j) with its constraint), G_w
// (n x n, ld n; Q = its first r columns), Sigma.
struct EntryAq {
    int n, m, r;
    const int *jk, *rptr, *rcol, *ridx;
    const double *Gw, *sig;
    double *Hm, *U, *YQ, *F;  // scratch: n * r, n * r, 2 n r, 2 n r
    EntryLp lp;
    // C = op(G_w) B for n x cols B and C (ld n), split over K where that pays: the
    // general form's products.  May use the caller's split-K workspaces.
    std::function<void(bool ta, int cols, const double* B, double* C)> product;
};

// out = a0 (AQ)^T u0 + a1 (AQ)^T u1 + add + ts sig .* vin  (d + lp.t entries; u1,
// add and vin may be null).
void entry_aqt(hipStream_t st, const EntryAq& q, const double* u0, double a0, const double* u1, double a1,
               const double* add, double ts, const double* vin, double* out);

// U = G_w H(v), which entry_aq_op reads.
void entry_form_u(hipStream_t st, const EntryAq& q, const double* v);

// With t = AQ v:
//   entry_aq_op:   out = (the symmetric M at the sampled pairs) + t.  lower: only M's
//                  entries with row >= col are valid; splits > 0: M is the sum of that
//                  many partial products n * n apart; M null: out += t instead.
//                  (The operator's LP part is not in t here.)  U is formed
//                  beforehand (entry_form_u), while M's partial products do not yet
//                  occupy the split-K workspace.
//   entry_aq_up:   z1 = ib (f - t);  rho = (f - t) - beta z1
//   entry_aq_up2:  z1 += ib (rho - t);  zout = zv + v
void entry_aq_op(hipStream_t st, const EntryAq& q, const double* M, bool lower, int splits, double* out);
void entry_aq_up(hipStream_t st, const EntryAq& q, const double* v, const double* f, double ib, double beta, double* z1,
                 double* rho);
void entry_aq_up2(hipStream_t st, const EntryAq& q, const double* v, const double* rho, double ib, double* z1,
                  const double* zv, double* zout);

}  // namespace wc
