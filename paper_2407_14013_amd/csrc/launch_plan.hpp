// Launch arithmetic of the split-K FP64 products (blas.hip), of the operator's
// forms for dense rows and entry sampling (dense_op.hip, entry_op.hip), of the
// batched solver (batched.hip) and of the Lanczos workgroup (lanczos.hip), free
// of HIP so that host code -- including host-compiled tests that enumerate
// shapes -- can evaluate it.  A split-K plan splits K into `splits` slices of kc
// values; the last slice takes the remainder klast = K - (splits - 1) kc, 1 <=
// klast <= kc, so slice s reads operand columns (or rows) s kc .. s kc + (its K)
// - 1 only.
#pragma once

#include <algorithm>

namespace wc {

// FP64 GEMM tiles (64 x 64 output, 16-deep K steps) and the split limits
constexpr int GBM = 64, GBN = 64, GBK = 16;
constexpr int GEMM_SPLITS = 8;        // most K-splits of a small product
constexpr int GEMM_SPLIT_TILES = 64;  // split K only below this many output tiles
constexpr int THIN_N = 16;            // most columns of the thin product
constexpr int THIN_LDS = 4096;        // doubles of B staged in LDS by the thin product
constexpr int THIN_SPLITS = 32;       // most K-splits of the thin split-K form

struct SplitPlan {
    int splits = 1;  // < 2: no split
    int kc = 0;      // K of every slice but the last
    int klast = 0;   // K of the last slice
};

inline long plan_cdiv(long a, long b) { return (a + b - 1) / b; }

// Square-tile product C (m x n) over K split in the z dimension: only for few
// output tiles (< max_tiles of gbm x gbn) and k >= 64; slices are multiples of
// gbk; at most max_splits, and splits m n partial products must fit in ws_len.
inline SplitPlan dgemm_split_plan(int m, int n, int k, long ws_len, int gbm, int gbn, int gbk, int max_splits,
                                  int max_tiles) {
    SplitPlan p;
    const long tiles = plan_cdiv(m, gbm) * plan_cdiv(n, gbn);
    if (tiles >= max_tiles || k < 64 || m <= 0 || n <= 0) return p;
    int splits = static_cast<int>(std::min<long>(max_splits, std::min<long>(plan_cdiv(k, 32), plan_cdiv(128, tiles))));
    if (splits < 2) return p;
    const int kc = static_cast<int>(plan_cdiv(plan_cdiv(k, splits), gbk) * gbk);
    splits = static_cast<int>(plan_cdiv(k, kc));
    if (splits < 2 || (long)splits * m * n > ws_len) return p;
    p.splits = splits;
    p.kc = kc;
    p.klast = k - (splits - 1) * kc;
    return p;
}

// Whether the 64 x 64 form issues its loads two K steps ahead of their use instead
// of one.  The second set of staging registers costs A B^T its fourth workgroup
// per CU (152 registers instead of 128), which counts where the launch has edge
// tiles, whose checked loads end it, and a fourth per CU to run beside them.
// C -= A B^T in us, two steps ahead and one: n = 1700, 729 workgroups, 227 and 237; n =
// 1800 330 and 310; n = 2000, k = 100 37.9 and 32.6; n = 3000, 2209 workgroups, 1143 and
// 1124; n = 4000, 3969 workgroups, 2464 and 2530; without edge tiles n = 2048 322 and
// 328.  The other products are faster two steps ahead, or the same, at every size
// (A^T B: n = 1800 306 and 308, n = 3000 1057 and 1121).
constexpr bool two_steps_ahead(bool ta, bool tb, bool edges, long workgroups) {
    return ta || !tb || !edges || workgroups <= 3 * 256 || workgroups > 12 * 256;
}

// Thin product (n <= 16 columns) with B staged in LDS: enough slices that a
// slice's kc x n block of B fits in thin_lds doubles and, with a workspace,
// about 2048 workgroups of 64 rows are in flight; at most max_splits.
inline SplitPlan thin_split_plan(int m, int n, int k, bool have_ws, long thin_lds, int max_splits) {
    SplitPlan p;
    int splits = static_cast<int>(std::max<long>(1, plan_cdiv((long)k * n, thin_lds)));
    if (have_ws)
        splits = static_cast<int>(std::max<long>(splits, std::min(plan_cdiv(k, 128), plan_cdiv(2048, plan_cdiv(m, 64)))));
    splits = std::min(splits, max_splits);
    const int kc = static_cast<int>(plan_cdiv(k, splits));
    p.splits = static_cast<int>(plan_cdiv(k, kc));
    p.kc = kc;
    p.klast = k - (p.splits - 1) * kc;
    return p;
}

// How many of nv vectors' products of r columns each one launch takes: all while
// their columns together are few enough for the thin product, else one by one
// (past THIN_N columns only the general product is left, whose few tiles need a
// split over K to fill the chip).  A preconditioner product at n = 2000, r = 9: 770
// us joined, 743 one by one; at n = 1000, r = 17: 755 us joined and not split over K,
// 580 one by one and split.
constexpr int thin_vectors(int r, int nv) { return r * nv <= THIN_N ? nv : 1; }

// Dense rows: whether the operator takes its off-diagonal blocks from the explicit
// script-A script-Q (m x d, read once each way) or as products with G_w.  The
// products cost some forty microseconds of launches whatever m d is, the explicit
// passes 16 m d bytes, from the last-level cache while both copies fit in it.
// newton_apply in us, explicit and products: n = 100, r = 60, m d = 17e6 116 and 124; n
// = 150, r = 20, m d = 25e6 347 and 322; n = 200, r = 10, 12e6 358 and 402, r = 15, 26e6
// 545 and 571, r = 20, 46e6 773 and 680; n = 300, r = 10, 27e6 1153 and 1119.
constexpr bool dense_explicit(long m, long d) { return m * d <= 20'000'000; }

// Entry sampling's latency-bound forms (entry_op.hip): where they are the faster
// ones, and H (n r doubles) fits in LDS.  precond_apply in us, these forms and the
// general ones: r = 4 70 and 91 at n = 512, 111 and 111 at n = 1024, 137 and 128 at n =
// 1200; r = 8, whose kernels hold EN_R columns and load a step at a time, 110 and
// 142 at n = 300, 173 and 174 at n = 640, 199 and 187 at n = 768, 269 and 230 at n = 1024.
constexpr int EN_R = 16;  // most columns of Q in one launch
constexpr bool entry_small(int n, int r) { return n <= (r <= 4 ? 1024 : 640) && r <= EN_R && n * r <= 8192; }

// The batched solver's pass settings for an instance without a tuning: packed rows
// that a wave streams at once and the edge of its MFMA tiles.  Up to n = 32 the
// 32 x 32 tiles are at most one for eight waves, and a packed row is short (528
// entries at n = 32).  Four iterations of 32 instances in ms, 4 rows with 16 x 16
// tiles and 2 rows with 32 x 32: n = 16 26.3 and 27.1, n = 32 38.1 and 39.5, n = 33 46.9
// and 45.8, n = 40 53.6 and 47.8, n = 47 81.2 and 75.7, n = 72 208 and 189.
struct BatchForm {
    int rows_per_wave, gemm_tile;
};
constexpr BatchForm batch_form(int n) { return n <= 32 ? BatchForm{4, 16} : BatchForm{2, 32}; }

// The Lanczos workgroup's split of w = T q: every row in nch chunks of clen
// columns (the last one shorter), thread t < n nch on row t % n and chunk t / n;
// one chunk where a row leaves no thread for a second.  Chunks have LZ_CHUNK
// columns at least: shorter ones cost more in the sum over them than they save.  A
// call in us, as many chunks as there are threads for, 8 columns at least and 16: n =
// 22 243, 194, 196; n = 32 414, 287, 288 (364 with one thread per row in the
// reorthogonalisation); n = 64 516, 444, 417; n = 100 626, 616, 571; n = 200 867, 862, 854.
// Its dynamic LDS in doubles: q (n, then LZ_TREG zeros, which a thread's
// register columns past the row's end are multiplied with: cl0 + u <= n - 1 +
// LZ_TREG - 1), w (n) at `w`, partial sums (n nch) at `pp`, the basis at `Q`.
constexpr int LZ_THREADS = 1024;
constexpr int LZ_TREG = 24;   // columns of its chunk of T that a thread keeps in registers
constexpr int LZ_CHUNK = 16;  // columns of a chunk at least

struct LanczosPlan {
    int nch, clen;
    int w, pp, Q;
};

constexpr LanczosPlan lanczos_plan(int n) {
    LanczosPlan p{};
    const int most = n > LZ_THREADS / 2 ? 1 : std::min(LZ_THREADS / n, (n + LZ_CHUNK - 1) / LZ_CHUNK);
    p.clen = (n + most - 1) / most;
    p.nch = (n + p.clen - 1) / p.clen;
    p.w = n + LZ_TREG;
    p.pp = p.w + n;
    p.Q = p.pp + (p.nch > 1 ? LZ_THREADS : 0);
    return p;
}

}  // namespace wc
