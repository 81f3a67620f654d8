"""Launches counted in the GEMM class of the event timings, form by form of the operator."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from paper_2407_14013_amd import Context  # noqa: E402
from paper_2407_14013_amd import _lib as L  # noqa: E402


# Y E and E (Y E) are GEMM launches whether or not the second one's partial
# products are summed (split over K at n = 100 and 300); entry sampling's general
# form (n = 1100) adds the products for U and F, its forms for small n none; dense
# rows with n <= 64 take E Y E in one kernel
@pytest.mark.parametrize("kind, n, gemms", [("dense", 40, 0), ("dense", 100, 2), ("entry", 300, 2), ("entry", 1100, 4)])
def test_gemm_class_counts_every_gemm_of_the_operator(kind, n, gemms):
    p = workloads.gaussian_sensing(n, 2, 4 * n, seed=n) if kind == "dense" else workloads.matrix_completion(n, 2, 20 * n, seed=n)
    with Context(p, rank_fixed=2) as ctx:
        x = torch.ones(ctx.aug_dim(), dtype=torch.float64, device="cuda")
        ctx.profile_enable([L.SDP_K_GEMM, L.SDP_K_SANDWICH])
        for _ in range(3):
            ctx.newton_apply(x)
        assert ctx.profile_get(L.SDP_K_GEMM)["launches"] == 3 * gemms
        assert ctx.profile_get(L.SDP_K_SANDWICH)["launches"] == (3 if kind == "dense" and n <= 64 else 6)
