"""The FP64 vector-unit round kernel's row sums (coefficients by row broadcast,
Chebyshev basis) at the edges of their groups of four and sixteen modes and of the
kernel's mode tiers, one, two and four paths per lane, both estimator forms, whole
and chunked slabs: increments against the FP64 oracle on the same Philox words,
1e-12 of the iterate as in the other parity tests."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,ns,kw", [
    (2, 1, 2, {}), (2, 2, 1, {}), (2, 3, 4, {}), (2, 6, 2, {}), (2, 7, 1, {}),          # P = 3, 4, 5, 8, 9
    (2, 10, 2, {}), (2, 11, 1, {}), (2, 14, 4, {}), (2, 15, 2, {}),                     # 12, 13, 16, 17
    (2, 18, 1, {}), (2, 19, 2, {}), (2, 26, 1, {}), (2, 27, 2, {}),                     # 20, 21, 28, 29
    (2, 30, 1, dict(estimator="picard")), (2, 12, 1, dict(estimator="picard")),
    (1, 13, 2, {}), (1, 30, 4, {}), (1, 15, 1, dict(estimator="picard", quad="ball")),
    (3, 2, 2, {}), (3, 7, 1, {}), (3, 11, 2, {}), (4, 3, 1, {}), (5, 2, 2, {})])
def test_fp64_rows_match_the_oracle(dim, n, ns, kw):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] fp64 rows", dim, n, ns, kw, flush=True)
    wl = W.small(dim=dim, n=n, M_deg=1, M=9 if dim < 3 else 2, T=0.3, f="sin", src="longtime", nstar=25, **kw)
    U = np.random.default_rng(n).standard_normal((1, wl.nsp, 2)) * 0.4
    with H.Plan(wl) as plan:
        plan.hpsmc_set_option("sample_1d", 0)
        plan.hpsmc_set_launch(ns, 4, 2, 20)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 1)
        got = plan.hpsmc_get_nodes(0)[0]
        steps = plan.hpsmc_stats()["path_steps"]
    ref, _, so = O.Problem(wl).iterate(U[0].reshape(-1), iter_tag=1)
    assert steps == so
    assert np.max(np.abs(got - ref.reshape(wl.nsp, 2))) <= 1e-12 * max(1.0, np.max(np.abs(ref)))
