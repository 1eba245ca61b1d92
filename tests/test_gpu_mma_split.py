"""The split half-precision products of the 2-D matrix-core kernel (P >= 17)
against the vector-unit kernel on the same Philox words: mode counts at the
edges of its blocks of eight and of the dispatch between FP32 and split
products, nodal values of very small and large magnitude (the power-of-two scale
of the tables), ball points outside the domain (the scale of the basis values,
and the vector-unit kernel where none fits), and non-finite nodal values.

Both kernels sum P^2 products in FP32; their path values differ by the rounding
of those sums, bounded as in the other matrix-core tests by 1e-4 of the largest
path value."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(wl, U, mma, **want):
    from paper_2608_22190_amd import hpsmc as H
    with H.Plan(wl) as plan:
        plan.hpsmc_set_option("sample_mfma", mma)
        plan.hpsmc_set_launch(1, 4, 2, 64)
        active = plan.hpsmc_get_option("sample_mfma_active")
        plan.hpsmc_set_probe(4)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 1)
        return plan.hpsmc_get_probe(0)[0], plan.hpsmc_get_increment(0)[0], plan.hpsmc_stats(), active


@pytest.mark.parametrize("n,scale,estimator", [
    (14, 1.0, "residual"), (15, 1.0, "residual"), (16, 1e-9, "residual"), (16, 1e6, "picard"), (17, 1.0, "picard"),
    (22, 1.0, "residual"), (23, 1e-20, "residual"), (30, 1e12, "residual")])
def test_split_products_match_the_vector_kernel(n, scale, estimator):
    print("[case] split", n, scale, estimator, flush=True)
    wl = W.small(dim=2, n=n, M_deg=3, M=37, T=0.5, f="affine", f_param=[0.7, 0.0, 0, 0], src="none", ic="singular",
                 precision="fp32", estimator=estimator, nstar=150)
    U = scale * np.random.default_rng(n).standard_normal((1, wl.nsp, 4))
    pm, em, sm, am = _run(wl, U, 1)
    pv, ev, sv, av = _run(wl, U, 0)
    assert (am, av) == (1, 0)
    assert sm["path_steps"] == sv["path_steps"]
    assert np.max(np.abs(pm - pv)) <= 1e-4 * np.max(np.abs(pv))
    assert np.max(np.abs(em - ev)) <= 1e-4 * np.max(np.abs(pv))


@pytest.mark.parametrize("nstar,active", [(2000, 1), (200, 1), (3, 0)])
def test_ball_points_outside_the_domain(nstar, active):
    print("[case] split ball", nstar, flush=True)
    wl = W.small(dim=2, n=16, M_deg=2, M=33, T=0.5, f="sin", src="longtime", precision="fp32", quad="ball",
                 nstar=nstar)
    U = 0.3 * np.random.default_rng(5).standard_normal((1, wl.nsp, 3))
    pm, em, sm, am = _run(wl, U, 1)
    pv, ev, sv, _ = _run(wl, U, 0)
    assert am == active
    assert sm["path_steps"] == sv["path_steps"]
    assert np.max(np.abs(pm - pv)) <= 1e-4 * (1.0 + np.max(np.abs(pv)))


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_values_stay_visible(bad):
    print("[case] split non-finite", bad, flush=True)
    wl = W.small(dim=2, n=16, M_deg=2, M=20, T=0.5, f="sin", src="longtime", precision="fp32", nstar=20)
    U = np.zeros((1, wl.nsp, 3))
    U[0, 7, 1] = bad
    _, em, sm, am = _run(wl, U, 1)
    assert am == 1
    assert not np.all(np.isfinite(em))
    assert sm["status_flags"] & 1
