"""Sizes at which the one-workgroup Lanczos kernel splits its work differently."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2407_14013_amd import linalg as la  # noqa: E402

EPS = 2.0 ** -53


# one chunk (n <= 16), two of 9 columns (17), three (33, 48) and four, chunks that
# end with or before a thread's 24 register columns (n = 146 | 147, 156 | 157), the last split row
# (512 | 513), the last one-workgroup size (640 | 641).  Before it, the same
# kernel on a NaN matrix, which leaves NaN in the LDS of the workgroups that
# it ran on: nothing of that may reach the result.
# T has the eigenvalue -3 apart from the rest in [-1, 1], so the process
# converges to rounding within 24 steps.  Bound: sums of length n, ten a step,
# and the breakdown threshold of 1e-13, times the norm.
@pytest.mark.parametrize("n", [1, 2, 3, 16, 17, 20, 22, 23, 32, 33, 48, 49, 64, 71, 89, 146, 147, 156, 157, 341, 342, 512, 513,
                               640, 641])
def test_lanczos_split_edges(n):
    rng = np.random.default_rng(n + 77)
    V, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = rng.uniform(-1.0, 1.0, n)
    lam[rng.integers(n)] = -3.0
    T = (V * lam) @ V.T
    T = 0.5 * (T + T.T)
    ref = np.linalg.eigvalsh(T)[0]
    Td = la.to_dev(T)
    nan = la.to_dev(np.full((500, 500), np.nan))
    for _ in range(16):
        la.dlanczos_min_eig(nan)
    got = [la.dlanczos_min_eig(Td) for _ in range(4)]
    assert np.all(np.isfinite(got))
    assert np.abs(np.array(got) - ref).max() <= (10 * n * EPS + 1e-13) * 3.0
