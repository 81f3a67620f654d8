"""Edge sizes of the HIP kernels whose split or route depends on the size.

Each test compares against NumPy / the oracle's formulas with a bound for FP64
sums of the length involved (c * K * eps times the operands' size).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import nt, reform as rf  # noqa: E402
from paper_2407_14013_amd import Context, batched  # noqa: E402
from paper_2407_14013_amd import linalg as la  # noqa: E402

EPS = 2.0 ** -53


@pytest.mark.parametrize("n", [31, 32, 33, 48, 49, 208, 255, 256, 258, 289])
def test_jacobi_clustered_and_zero_columns(n):
    # block pairs with equal eigenvalues (rotation angles of 45 degrees and
    # none at all), a zero column (nothing to rotate) and padded columns: the
    # rounds past a sweep's first rotate only between the two blocks of a pair
    rng = np.random.default_rng(n)
    Q1, _ = np.linalg.qr(rng.standard_normal((n, n)))
    Q2, _ = np.linalg.qr(rng.standard_normal((n, n)))
    d = np.repeat([4.0, 1.0, 0.25], [n // 3, n // 3, n - 2 * (n // 3)])
    A = (Q1 * d) @ Q2.T
    A[:, n // 2] = 0.0
    Ad = la.to_dev(A)
    s, V, sweeps = la.djacobi_svd(Ad)
    s, Vg, Aout = s.cpu().numpy(), la.from_dev(V), la.from_dev(Ad)
    ref = np.linalg.svd(A, compute_uv=False)
    assert 1 <= sweeps <= 60  # the call's own limit: clusters converge slowly (28 to 43 sweeps past n = 200)
    assert np.abs(s - ref).max() <= 20 * n * EPS * ref[0]
    assert np.abs(Vg.T @ Vg - np.eye(n)).max() <= 20 * n * EPS
    assert np.abs(A @ Vg - Aout).max() <= 20 * n * EPS * ref[0]


# a round of two launches with A's and V's rows apart (n = 639: 20 pairs x 5 row
# chunks), together (705, 1024: 32 x 8 workgroups), and of three launches (1025),
# rows one past a chunk; with V and without
@pytest.mark.parametrize("n", [639, 705, 769, 1024, 1025])
def test_jacobi_large_round_forms(n):
    rng = np.random.default_rng(n)
    d = np.linspace(1.0, 3.0, n)
    A = np.linalg.qr(rng.standard_normal((n, n)))[0] * d + 1e-3 * rng.standard_normal((n, n))
    Ad = la.to_dev(A)
    s, V, sweeps = la.djacobi_svd(Ad)
    s, Vg, Aout = s.cpu().numpy(), la.from_dev(V), la.from_dev(Ad)
    ref = np.linalg.svd(A, compute_uv=False)
    assert 1 <= sweeps <= 60
    assert np.abs(s - ref).max() <= 20 * n * EPS * ref[0]
    assert np.abs(Vg.T @ Vg - np.eye(n)).max() <= 20 * n * EPS
    assert np.abs(A @ Vg - Aout).max() <= 20 * n * EPS * ref[0]
    s1, _, _ = la.djacobi_svd(la.to_dev(A), want_v=False)
    assert np.abs(s1.cpu().numpy() - ref).max() <= 20 * n * EPS * ref[0]


# script-A script-Q rows of 63..65, 126..129 and 255..257 entries (the register
# forms of the batched Krylov loop and the general one), n at the default
# tile's edge, odd numbers of packed pairs, and (rank_max 79) vectors that do
# not fit in LDS.  The bars are those of the workload's own checks: both solvers
# stop at a relative gap of 1e-8.
@pytest.mark.parametrize("n, r, rank_max", [(17, 1, 10), (22, 3, 10), (23, 3, 10), (33, 2, 10), (47, 3, 10), (48, 2, 10),
                                            (65, 2, 10), (86, 3, 10), (87, 3, 10), (80, 1, 79)])
@pytest.mark.parametrize("prec", [0, 1])
def test_batched_edges_match_single_solver(n, r, rank_max, prec):
    p = workloads.gaussian_sensing(n, r, min(3 * n * r, n * (n + 1) // 2), seed=n + 1000 * r)
    res, Xs, _ = batched.solve_batched([p], inner_prec=prec, rank_max=rank_max)
    with Context(p, rank_max=rank_max) as ctx:
        one = ctx.solve()
        X = ctx.get_point()[0]
    assert res[0]["status"] == 0
    assert abs(res[0]["pobj"] - one["pobj"]) <= 2e-8 * (1.0 + abs(one["pobj"]))
    Xstar = p["U"] @ p["U"].T
    for Y in (Xs[0], X):
        assert np.linalg.norm(Y.cpu().numpy() - Xstar) <= 1e-6 * np.linalg.norm(Xstar)


def scaled_point(n, seed):
    X, S = workloads.random_pd_pair(n, seed=seed, spread=0.5)
    G, _, _ = nt.nt_factor(X, S)
    return X, S, G @ G.T


# dense rows: the operator's single-workgroup middle (n <= 64, tile edges) and
# the split-K one, odd m and d, one constraint, vectors that are only 8-byte
# aligned.  1e-10 of the largest entry, the bound of the operator's other
# checks: FP64 sums of length n (n + 1) / 2 <= 2 211 and eigenvectors of
# well-separated spectra.
@pytest.mark.parametrize("n, m", [(2, 1), (3, 4), (15, 37), (16, 64), (17, 101), (48, 129), (63, 300), (64, 257),
                                  (65, 301), (66, 128), (97, 255)])
@pytest.mark.parametrize("rank", [1, 2])
def test_dense_operator_and_preconditioner_edges(n, m, rank):
    if rank >= n:
        pytest.skip("the rank parameter is below n")
    p = workloads.generic_sensing(n, m, seed=n + m)
    X, S, W = scaled_point(n, seed=n)
    sp = rf.eig_split(W, rank_fixed=rank)
    sig, E = rf.sigma_diag(sp), rf.e_matrix(sp)
    N = m + rf.dim_d(n, rank)
    x = np.random.default_rng(m).standard_normal(N)
    t, b = rf.aug_apply(p, sp, E, sig, x[:m], x[m:])
    ref = np.concatenate([t, b])
    for prec, tol in ((0, 1e-10), (1, 1e-5)):  # FP32: E Y E and the rows carry 24 bits, sums of length n in FP32
        with Context(p, rank_fixed=rank, inner_prec=prec) as ctx:
            ctx.set_point(*(torch.from_numpy(a).cuda() for a in (X, np.zeros(m), S)))
            assert ctx.aug_dim() == N
            for shift in (0, 1):
                buf = torch.zeros(N + shift, dtype=torch.float64, device="cuda")
                buf[shift:] = torch.from_numpy(x)
                out = torch.full((N + shift,), np.nan, dtype=torch.float64, device="cuda")
                got = ctx.newton_apply(buf[shift:], out[shift:], prec=prec if prec else None).cpu().numpy()
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (prec, shift)
            if prec == 0:
                # backward error of P z = x with the oracle's P
                P = rf.precond_matrix(rf.aq_matrix(p, sp), sp, sig, ctx.get_scaling()["beta"])
                z = ctx.precond_apply(torch.from_numpy(x).cuda()).cpu().numpy()
                assert np.abs(P @ z - x).max() <= 1e-9 * np.abs(P).sum(1).max() * np.abs(z).max()


# entry sampling: rows with no sampled entry, one pair, r at 4 | 5 and 16 | 17
# columns per launch, n at 1024 and n r at 8192 (the latency-bound forms' range),
# with and without the LP block.  The split is the GPU's own, so what is
# compared is sums of length n: 1e-10 of the largest entry as above.
@pytest.mark.parametrize("n, m, rank, lp", [(2, 1, 1, True), (5, 3, 2, False), (33, 200, 3, True), (64, 500, 4, True),
                                            (65, 500, 5, True), (130, 2000, 16, False), (130, 900, 17, True),
                                            (512, 300, 16, False), (513, 300, 16, False), (1024, 257, 1, True),
                                            (1025, 255, 2, True)])
@pytest.mark.parametrize("sampled", [0, 1])
def test_entry_operator_and_preconditioner_edges(n, m, rank, lp, sampled):
    rng = np.random.default_rng(n + m)
    p = workloads.robust_completion(n, m, min(m, 5), seed=n) if lp else workloads.matrix_completion(n, rank, m, seed=n)
    X, S = workloads.random_pd_pair(n, seed=n, spread=0.5)
    pts = [X, np.zeros(m), S]
    if lp:
        ell = len(p["lp"]["c"])
        pts += [np.exp(rng.standard_normal(ell)), np.exp(rng.standard_normal(ell))]
    with Context(p, rank_fixed=rank, sparse_sandwich=sampled) as ctx:
        ctx.set_point(*(torch.from_numpy(a).cuda() for a in pts))
        g = ctx.get_scaling()
        lam, V, r = g["lam"], g["V"].cpu().numpy(), g["r"]
        assert r == rank
        sp = {"n": n, "r": r, "tau": 0.5 * lam[r], "lam": lam, "V": V, "Q": V[:, :r], "Qp": V[:, r:],
              "lam_top": lam[:r], "lam_perp": lam[r:]}
        sig, E, AQ = rf.sigma_diag(sp), rf.e_matrix(sp), rf.aq_matrix(p, sp)
        N = ctx.aug_dim()
        x = rng.standard_normal(N)
        if lp:
            lsp = rf.lp_split(sp, ctx.lp_split()["w"].cpu().numpy(), cap=int(ctx.options.lp_top_max))
            ref = np.concatenate(rf.aug_apply_lp(p, sp, lsp, E, sig, x[:m], x[m:]))
            AQ, sig = rf.aq_matrix_lp(p, sp, lsp), np.concatenate([sig, lsp["sig"]])
        else:
            ref = np.concatenate(rf.aug_apply(p, sp, E, sig, x[:m], x[m:]))
        assert N == ref.size
        for shift in (0, 1):  # vectors that are only 8-byte aligned too
            buf = torch.zeros(N + shift, dtype=torch.float64, device="cuda")
            buf[shift:] = torch.from_numpy(x)
            got = ctx.newton_apply(buf[shift:]).cpu().numpy()
            assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
            z = ctx.precond_apply(buf[shift:]).cpu().numpy()
            # [beta I, AQ; AQ^T, -tau^2 Sigma] z = x
            Pz = np.concatenate([g["beta"] * z[:m] + AQ @ z[m:], AQ.T @ z[:m] - sp["tau"] ** 2 * sig * z[m:]])
            rows = np.concatenate([g["beta"] + np.abs(AQ).sum(1), np.abs(AQ).sum(0) + sp["tau"] ** 2 * sig])
            assert np.abs(Pz - x).max() <= 1e-9 * rows.max() * np.abs(z).max()


# panels: one row past a block, an outer panel's edges (256, 512 | 513), inverse
# blocks of 1024; the input's strict upper triangle is not read.  The bounds
# are those of the factorisation's other checks.
@pytest.mark.parametrize("n", [2, 30, 34, 63, 65, 96, 257, 289, 511, 514, 543, 769, 1023, 1025, 1060])
def test_cholesky_and_inverse_edges(n):
    rng = np.random.default_rng(n)
    M = rng.standard_normal((n, n))
    A = M @ M.T + n * np.eye(n)
    Ad = la.to_dev(np.where(np.triu(np.ones((n, n)), 1) > 0, np.nan, A))
    st, info = la.dpotrf(Ad)
    assert st == 0 and info == 0
    Lg, Lr = la.from_dev(Ad), np.linalg.cholesky(A)
    assert not np.triu(Lg, 1).any()
    assert np.abs(Lg - Lr).max() <= 50 * n * EPS * np.abs(Lr).max()
    Xg = la.from_dev(la.dtrtri(la.to_dev(np.where(np.triu(np.ones((n, n)), 1) > 0, np.nan, Lr))))
    ref = np.linalg.inv(Lr)
    assert not np.triu(Xg, 1).any()
    assert np.abs(Xg - ref).max() <= 100 * n * EPS * np.abs(ref).max()
    # a bad pivot in the first, a middle and the last column
    for j in (0, n // 2, n - 1):
        B = A.copy()
        B[j, j] = -1.0
        st, info = la.dpotrf(la.to_dev(B))
        assert st == -5 and info == j + 1


# 128 x 128 tiles by 16-byte LDS loads: K of 2 to one past a step, tiles with one
# pair of rows or columns, 160 tiles and fewer (the general form); the same
# operands 8 bytes further on take the general form and give the same bits.
# The bound is that of the product's other checks.
@pytest.mark.parametrize("ta", ["N", "T"])
@pytest.mark.parametrize("tb", ["N", "T"])
@pytest.mark.parametrize("m, n, k", [(4096, 4098, 2), (4098, 4096, 14), (4096, 4100, 16), (4226, 3970, 18),
                                     (4100, 4100, 46), (4098, 4098, 130), (1666, 1602, 50), (2048, 1280, 34),
                                     (1536, 1536, 34), (2049, 1801, 33)])
def test_gemm_lds_loads_match_the_general_form(ta, tb, m, n, k):
    rng = np.random.default_rng(m + n + k)
    A = rng.standard_normal((k, m) if ta == "T" else (m, k))
    B = rng.standard_normal((n, k) if tb == "T" else (k, n))
    ref = (A.T if ta == "T" else A) @ (B.T if tb == "T" else B)

    def shifted(a):
        d = la.to_dev(a)
        buf = torch.full((d.numel() + 1,), np.nan, dtype=torch.float64, device="cuda")
        buf[1:] = d.flatten()
        return buf[1:].view(d.shape)

    got = [torch.full((n, m), np.nan, dtype=torch.float64, device="cuda") for _ in range(2)]
    la.dgemm(ta, tb, 1.0, la.to_dev(A), la.to_dev(B), 0.0, got[0])
    la.dgemm(ta, tb, 1.0, shifted(A), shifted(B), 0.0, got[1])
    assert np.abs(la.from_dev(got[0]) - ref).max() <= 4 * k * EPS * np.abs(A).max() * np.abs(B).max()
    assert torch.equal(got[0], got[1])


# the sampled products against the dense ones: 8, 4 and 2 staged columns (n = 2048
# | 2049, 4096 | 4097), fewer slabs than XCDs, a last slab of one row, one pair,
# more pairs than a workgroup holds at a time.  Sums of n products in another
# order, of entries of E that cancel: 1e-10 of the largest, as above.
@pytest.mark.parametrize("n, m", [(70, 1), (129, 2000), (577, 166000), (2048, 3000), (2049, 60000), (4097, 300000)])
def test_sampled_products_match_the_dense_ones(n, m):
    rng = np.random.default_rng(n)
    p = workloads.matrix_completion(n, 2, m, seed=n)
    d = np.exp(0.5 * rng.standard_normal((2, n)))
    U = rng.standard_normal((n, 2)) / np.sqrt(n)
    pts = [np.diag(d[0]) + U @ U.T, np.zeros(m), np.diag(d[1])]
    x = None
    got = []
    for sampled in (0, 1):
        with Context(p, rank_fixed=2, sparse_sandwich=sampled) as ctx:
            ctx.set_point(*(torch.from_numpy(a).cuda() for a in pts))
            if x is None:
                x = torch.from_numpy(rng.standard_normal(ctx.aug_dim())).cuda()
            got.append(ctx.newton_apply(x).cpu().numpy())
    assert np.abs(got[1] - got[0]).max() <= 1e-10 * np.abs(got[0]).max()


# results stored four rows at a time, and one by one where the result is only
# aligned to its own type: the same bits (256 x 256 BF16 tiles and the 128 x 128
# ones of both types, ragged edges)
@pytest.mark.parametrize("prec, m, n", [(1, 1032, 1030), (2, 1032, 1030), (2, 3896, 3620)])
@pytest.mark.parametrize("out_kind", [0, 1, 2, 3])
def test_low_precision_stores_do_not_depend_on_alignment(prec, m, n, out_kind):
    rng = np.random.default_rng(m + n)
    M = rng.standard_normal((m, m))
    A = la.to_lowp(la.to_dev(M + M.T), prec)
    B = la.to_lowp(la.to_dev(rng.standard_normal((m, n))), prec)
    dt = {0: torch.float32, 1: torch.int16, 2: torch.float64, 3: torch.float64}[out_kind]
    got = []
    for shift in (0, 1):
        buf = torch.ones(m * n + 1, dtype=dt, device="cuda")
        Cm = buf[shift:shift + m * n].view(n, m)
        got.append(la.gemm_lp_sym(prec, out_kind, A, B, Cm).clone())
        assert buf[m * n if shift == 0 else 0].item() == 1  # nothing past the result
    assert torch.equal(got[0], got[1])


# staging: instances of 33 MB (a group of its own each) between small ones, in an
# order that mixes both, against each instance staged alone; two iterations, so
# rounding has not grown: 1e-9 as for the operator's other comparisons
def test_batched_staging_groups_match_single_instances():
    sizes = [(16, 48), (96, 900), (17, 60), (96, 901), (20, 100), (24, 216), (95, 899), (2, 1)]
    probs = [workloads.gaussian_sensing(n, 1, m, seed=n + m) for n, m in sizes]
    res, Xs, ys = batched.solve_batched(probs, want_y=True, max_ipm_iter=2)
    for p, r, X, y in zip(probs, res, Xs, ys):
        one, X1, y1 = batched.solve_batched([p], want_y=True, max_ipm_iter=2)
        assert r["iterations"] == one[0]["iterations"]
        assert abs(r["pobj"] - one[0]["pobj"]) <= 1e-9 * (1.0 + abs(one[0]["pobj"]))
        assert (X - X1[0]).abs().max() <= 1e-9 * X1[0].abs().max()
        assert (y - y1[0]).abs().max() <= 1e-9 * (1.0 + y1[0].abs().max())
    bad = [dict(p) for p in probs]
    bad[4] = dict(bad[4], A=np.where(np.arange(bad[4]["A"].size).reshape(bad[4]["A"].shape) == 7, np.inf, bad[4]["A"]))
    with pytest.raises(Exception, match="non-finite"):
        batched.solve_batched(bad, max_ipm_iter=2)


# K of one to six 16-deep steps, whole and one more: where the loop that loads
# two steps ahead ends; interior and edge tiles.  The bound of the product's
# other checks.
@pytest.mark.parametrize("ta", ["N", "T"])
@pytest.mark.parametrize("tb", ["N", "T"])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97])
def test_small_tile_gemm_step_counts(ta, tb, k):
    m, n = 600, 577  # 100 tiles of 64 x 64: no split over K
    rng = np.random.default_rng(k)
    A = rng.standard_normal((k, m) if ta == "T" else (m, k))
    B = rng.standard_normal((n, k) if tb == "T" else (k, n))
    C0 = rng.standard_normal((m, n))
    ref = 1.5 * (A.T if ta == "T" else A) @ (B.T if tb == "T" else B) - 0.5 * C0
    Cd = la.to_dev(C0)
    la.dgemm(ta, tb, 1.5, la.to_dev(A), la.to_dev(B), -0.5, Cd)
    bound = 4 * k * EPS * (np.abs(A).max() * np.abs(B).max() * 1.5 + 0.5 * np.abs(C0).max())
    assert np.abs(la.from_dev(Cd) - ref).max() <= bound + EPS * np.abs(ref).max()
