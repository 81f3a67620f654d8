"""Dense rows on both sides of the rule for the off-diagonal blocks.

m d = 18.4e6 takes the explicit script-A script-Q, 23.5e6 and 22.6e6 (odd n and m) the
products with G_w.  1e-10 of the largest entry against the oracle, the bound of
the operator's other checks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import nt, reform as rf  # noqa: E402
from paper_2407_14013_amd import Context  # noqa: E402


@pytest.mark.parametrize("n, m, rank", [(99, 4950, 50), (98, 4851, 97), (97, 4753, 96)])
def test_operator_at_large_ranks(n, m, rank):
    p = workloads.generic_sensing(n, m, seed=n)
    X, S = workloads.random_pd_pair(n, seed=n, spread=0.5)
    G, _, _ = nt.nt_factor(X, S)
    sp = rf.eig_split(G @ G.T, rank_fixed=rank)
    x = np.random.default_rng(m).standard_normal(m + rf.dim_d(n, rank))
    ref = np.concatenate(rf.aug_apply(p, sp, rf.e_matrix(sp), rf.sigma_diag(sp), x[:m], x[m:]))
    with Context(p, rank_fixed=rank) as ctx:
        ctx.set_point(*(torch.from_numpy(a).cuda() for a in (X, np.zeros(m), S)))
        assert ctx.aug_dim() == x.size
        for shift in (0, 1):  # vectors that are only 8-byte aligned too
            buf = torch.zeros(x.size + shift, dtype=torch.float64, device="cuda")
            buf[shift:] = torch.from_numpy(x)
            got = ctx.newton_apply(buf[shift:]).cpu().numpy()
            assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
