"""The tabulated lattice form of the 1-D FP64 rounds against the general kernel
on the same Philox words: lattice points that fall on the boundary (exit at
|X| = 1 exactly), several rounds with paths carried over, rows wide enough to
shrink the LDS window, one to four paths per lane, several instances, intervals
and sample slices of a wave and less, and the mode counts on both sides of the
dispatch.  The residual is taken at x_j + m J instead of at the position's
accumulated sum, which differ by about 1e-15 times the square root of the steps:
1e-12 of the largest path value, the bar of the parity tests; the exits and so
the evaluation counts are the same."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(wl, win, launch, U):
    from paper_2608_22190_amd import hpsmc as H
    with H.Plan(wl) as plan:
        plan.hpsmc_set_option("sample_1d", win)
        plan.hpsmc_set_launch(*launch)
        plan.hpsmc_set_probe(min(wl.M, 5))
        for iv, u in enumerate(U):
            plan.hpsmc_set_nodes(iv, u)
        plan.hpsmc_reset_stats()
        if wl.schedule == "sweeps":
            plan.hpsmc_sweep(1)
        else:
            plan.hpsmc_iterate(0, 1)
        n_iv = len(wl.degree) if wl.schedule == "sweeps" else 1
        return ([plan.hpsmc_get_probe(iv) for iv in range(n_iv)], [plan.hpsmc_get_increment(iv)[0] for iv in range(n_iv)],
                plan.hpsmc_stats()["path_steps"])


@pytest.mark.parametrize("n,deg,M,T,nstar,launch,kw", [
    (3, 1, 200, 0.5, 4, (1, 4, 2, 64), {}),               # J = 1/2 and x = 0: points on the boundary
    (1, 2, 64, 0.125, 100, (2, 4, 8, 64), {}),            # J = 1/20
    (6, 4, 65, 0.5, 200, (2, 4, 8, 256), {}),
    (5, 2, 130, 0.5, 2500, (4, 4, 2, 256), {}),           # three rounds
    (3, 1, 40, 0.5, 60000, (1, 4, 4, 256), {}),           # wide rows: eight steps a window
    (18, 3, 300, 0.3, 700, (1, 2, 3, 64), dict(src="none", ic="singular")),   # 20 modes, the last tabulated
    (19, 3, 300, 0.3, 700, (1, 2, 3, 64), dict(src="none", ic="singular")),   # 21: evaluated
    (4, [2, 3, 1], 33, 0.6, 90, (2, 4, 2, 64), dict(n_intervals=3, schedule="sweeps", n_instances=3)),
    (8, 2, 1, 0.5, 3000, (1, 4, 2, 64), {})])             # one path a node
def test_lattice_form_matches_the_general_kernel(n, deg, M, T, nstar, launch, kw):
    print("[case] lattice", n, deg, M, T, nstar, launch, kw, flush=True)
    wl = W.small(dim=1, n=n, M_deg=deg, M=M, T=T, f="sin", nstar=nstar, precision="fp64", **kw)
    rng = np.random.default_rng(n)
    U = [rng.standard_normal((wl.n_instances, wl.nsp, m + 1)) * 0.4 for m in wl.degree]
    pg, eg, sg = _run(wl, 0, launch, U)
    pl, el, sl = _run(wl, 1, launch, U)
    assert sl == sg
    for a, b, c, d in zip(pl, pg, el, eg):
        scale = 1.0 + np.max(np.abs(b))
        assert np.max(np.abs(a - b)) <= 1e-12 * scale
        assert np.max(np.abs(c - d)) <= 1e-12 * scale
