"""Edge sizes of the HIP kernels whose split or route depends on the size.

Each test compares against NumPy / the oracle's formulas with a bound for FP64
sums of the length involved (c * K * eps times the operands' size).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
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
