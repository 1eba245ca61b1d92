"""The ball rule with jumps so long that the basis values at ball points outside the
domain exceed the half-precision range (P >= 17): the rounds stay on the matrix
cores, with FP32 products.  On both sides of the line, both forms of the estimator,
against the vector-unit kernel on the same words to the 1e-4 bound of the other
matrix-core tests (the sums' rounding, relative to the largest path value)."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(wl, U, mma, active):
    from paper_2608_22190_amd import hpsmc as H
    with H.Plan(wl) as plan:
        plan.hpsmc_set_option("sample_mfma", mma)
        plan.hpsmc_set_launch(1, 4, 2, 64)
        assert plan.hpsmc_get_option("sample_mfma_active") == active
        plan.hpsmc_set_probe(4)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 1)
        return plan.hpsmc_get_probe(0)[0], plan.hpsmc_get_increment(0)[0], plan.hpsmc_stats()["path_steps"]


# log2 of twice the largest basis value: 14.7 (halves), 16.4, 19.0, 18.0, 24.3 (FP32), 25.6 (vector units)
@pytest.mark.parametrize("n,nstar,active", [(15, 45, 1), (15, 29, 1), (16, 20, 1), (30, 300, 1), (24, 36, 1), (24, 29, 0)])
@pytest.mark.parametrize("estimator", ["residual", "picard"])
def test_long_jumps_stay_on_the_matrix_cores(n, nstar, active, estimator):
    print("[case] ball long jumps", n, nstar, estimator, flush=True)
    wl = W.small(dim=2, n=n, M_deg=2, M=21, T=0.5, f="affine", f_param=[0.7, 0.0, 0, 0], src="longtime", precision="fp32",
                 quad="ball", nstar=nstar, estimator=estimator)
    U = 0.3 * np.random.default_rng(5).standard_normal((1, wl.nsp, 3))
    pm, em, sm = _run(wl, U, 1, active)
    pv, ev, sv = _run(wl, U, 0, 0)
    assert sm == sv
    assert np.max(np.abs(pm - pv)) <= 1e-4 * (1.0 + np.max(np.abs(pv)))
    assert np.max(np.abs(em - ev)) <= 1e-4 * (1.0 + np.max(np.abs(pv)))
