"""The fractional kernel's waves: items dealt out over several passes of the grid, one to
four waves a block, paths carried over many short rounds, slab rows of more than 64
entries and source series longer than a row.  FP64 against the oracle to the 1e-12 of the
other fractional tests; FP32 at the discrete space's exact fixed point, where every
path's residual is rounding alone, to the 2e-5 of that test."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha,n,deg,M,src,launch,kw", [
    (0.7, 3, 2, 9000, "frac_longtime", (1, 1, 1, 64), {}),          # 844 items, 256 waves: four passes
    (0.4, 4, 3, 11000, "frac_longtime", (1, 2, 1, 16), {}),         # five passes, four rounds
    (1.3, 32, 1, 5, "frac_longtime", (1, 4, 2, 20), {}),            # the longest rows
    (0.4, 5, 2, 70, "frac_singular", (1, 3, 1, 16), dict(src_param=[0.51, 0, 0, 0, 0, 0, 0, 0])),
    (1.7, 6, 2, 65, "none", (1, 4, 1, 16), dict(ic="nodal", ic_data=np.zeros((1, 6)))),
    (1.0, 31, 1, 3, "frac_poly", (1, 4, 4, 20), dict(src_param=[0.5, -0.3, 0.2, 0.7, 0, 0, 0, 0], estimator="picard"))])
def test_items_rows_and_rounds_fp64(alpha, n, deg, M, src, launch, kw):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] frac waves", alpha, n, deg, M, src, launch, flush=True)
    wl = W.small(dim=1, n=n, M_deg=deg, M=M, T=0.3, f="u_minus_u3", src=src, alpha=alpha, nstar=53, **kw)
    U = np.random.default_rng(n).standard_normal((1, n, deg + 1)) * 0.4
    with H.Plan(wl) as plan:
        plan.hpsmc_set_launch(*launch)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 2)
        got = plan.hpsmc_get_nodes(0)[0]
        steps = plan.hpsmc_stats()["path_steps"]
    Uo, _, so = O.Problem(wl).iterate(U[0].reshape(-1), iter_tag=2)
    assert steps == so
    assert np.max(np.abs(got - Uo.reshape(n, deg + 1))) <= 1e-12 * max(1.0, np.max(np.abs(Uo)))


@pytest.mark.parametrize("alpha,launch", [(0.1, (1, 1, 1, 16)), (0.4, (1, 4, 4, 128)), (1.0, (1, 2, 1, 20)), (1.9, (1, 4, 2, 64))])
def test_fixed_point_fp32(alpha, launch):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] frac fixed point fp32", alpha, launch, flush=True)
    wl = W.small(dim=1, n=5, M_deg=2, M=4000, T=0.5, f="u_minus_u3", src="frac_poly", alpha=alpha, precision="fp32",
                 src_param=[0.5, -0.3, 0.2, 0.7, 0, 0, 0, 0])
    pb = O.Problem(wl)
    x, t = pb.grid(0)
    U = np.array([[[pb.exact([xj], tl) for tl in t] for xj in x]])
    with H.Plan(wl) as plan:
        plan.hpsmc_set_launch(*launch)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 0)
        eps, _ = plan.hpsmc_get_increment(0)
        assert plan.hpsmc_stats()["path_steps"] > 0
    assert np.max(np.abs(eps)) < 2e-5
