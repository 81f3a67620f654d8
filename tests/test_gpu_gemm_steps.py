"""A B^T in 64 x 64 tiles with its loads issued one K step ahead (784 workgroups, edge tiles).

K of one step, whole and one more or less, up to four; C scaled and added, and
not read; the bound of the product's other checks.  The same product over fewer
columns runs two steps ahead and gives the same bits.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2407_14013_amd import linalg as la  # noqa: E402

EPS = 2.0 ** -53


@pytest.mark.parametrize("k", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65])
@pytest.mark.parametrize("beta", [0.0, -0.5])
def test_one_step_ahead(k, beta):
    m, n = 1780, 1777
    rng = np.random.default_rng(k)
    A, B, C0 = rng.standard_normal((m, k)), rng.standard_normal((n, k)), rng.standard_normal((m, n))
    ref = 1.5 * A @ B.T + beta * C0
    Cd = la.to_dev(C0 if beta else np.full_like(C0, np.nan))
    Ad, Bd = la.to_dev(A), la.to_dev(B)
    la.dgemm("N", "T", 1.5, Ad, Bd, beta, Cd)
    bound = 4 * k * EPS * (np.abs(A).max() * np.abs(B).max() * 1.5 + abs(beta) * np.abs(C0).max())
    assert np.abs(la.from_dev(Cd) - ref).max() <= bound + EPS * np.abs(ref).max()
    few = 64 * 20  # 560 workgroups
    Cf = la.to_dev(C0[:, :few])
    la.dgemm("N", "T", 1.5, Ad, la.to_dev(B[:few]), beta, Cf)
    assert torch.equal(Cf, Cd[:few])
