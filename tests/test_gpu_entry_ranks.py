"""Entry sampling at ranks where its products take another form.

Eight columns of Q and nine (two vectors in one thin product, or one each),
sixteen and seventeen (the thin product and the general one, whose split-K
workspace the operator's own partial products take at n = 300), n at the edges of
the latency-bound forms (640 | 641 for r > 4, 1024 | 1025 below), with and without
the LP block.  The split is the GPU's own, so what is compared is sums of
length n: 1e-10 of the largest entry, the bound of the operator's other checks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import reform as rf  # noqa: E402
from paper_2407_14013_amd import Context  # noqa: E402


@pytest.mark.parametrize("n, m, rank, lp", [(300, 400, 17, True), (640, 300, 10, False), (641, 300, 10, True),
                                            (640, 200, 5, True), (641, 200, 5, False), (820, 150, 9, False),
                                            (1024, 200, 4, False), (1025, 200, 8, True), (1025, 200, 9, True),
                                            (1025, 150, 16, False), (1025, 150, 17, True)])
def test_products_at_the_ranks_where_their_form_changes(n, m, rank, lp):
    rng = np.random.default_rng(n + rank)
    p = workloads.robust_completion(n, m, 5, seed=n) if lp else workloads.matrix_completion(n, rank, m, seed=n)
    X, S = workloads.random_pd_pair(n, seed=n, spread=0.5)
    pts = [X, np.zeros(m), S]
    if lp:
        ell = len(p["lp"]["c"])
        pts += [np.exp(rng.standard_normal(ell)), np.exp(rng.standard_normal(ell))]
    with Context(p, rank_fixed=rank) as ctx:
        ctx.set_point(*(torch.from_numpy(a).cuda() for a in pts))
        g = ctx.get_scaling()
        lam, V, r = g["lam"], g["V"].cpu().numpy(), g["r"]
        assert r == rank
        sp = {"n": n, "r": r, "tau": 0.5 * lam[r], "lam": lam, "V": V, "Q": V[:, :r], "Qp": V[:, r:],
              "lam_top": lam[:r], "lam_perp": lam[r:]}
        sig, E, AQ = rf.sigma_diag(sp), rf.e_matrix(sp), rf.aq_matrix(p, sp)
        x = rng.standard_normal(ctx.aug_dim())
        if lp:
            lsp = rf.lp_split(sp, ctx.lp_split()["w"].cpu().numpy(), cap=int(ctx.options.lp_top_max))
            ref = np.concatenate(rf.aug_apply_lp(p, sp, lsp, E, sig, x[:m], x[m:]))
            AQ, sig = rf.aq_matrix_lp(p, sp, lsp), np.concatenate([sig, lsp["sig"]])
        else:
            ref = np.concatenate(rf.aug_apply(p, sp, E, sig, x[:m], x[m:]))
        got = ctx.newton_apply(torch.from_numpy(x).cuda()).cpu().numpy()
        assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
        z = ctx.precond_apply(torch.from_numpy(x).cuda()).cpu().numpy()
        # [beta I, AQ; AQ^T, -tau^2 Sigma] z = x
        Pz = np.concatenate([g["beta"] * z[:m] + AQ @ z[m:], AQ.T @ z[:m] - sp["tau"] ** 2 * sig * z[m:]])
        rows = np.concatenate([g["beta"] + np.abs(AQ).sum(1), np.abs(AQ).sum(0) + sp["tau"] ** 2 * sig])
        assert np.abs(Pz - x).max() <= 1e-9 * rows.max() * np.abs(z).max()
