"""The tables of half-precision parts that the matrix-core kernels read, written 16 steps
and two modes at a time: step counts around 16, the lowest and highest temporal degrees,
a polynomial source in the table, unequal blocks of several intervals, and an image of
many entry parts (5-D, P = 10).  Against the vector-unit kernel on the same Philox words
to the 1e-4 bound of the other matrix-core tests, which is their FP32 sums' rounding."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,deg,nstar,kw", [
    (2, 16, 1, 1, {}), (2, 15, 7, 15, {}), (2, 16, 31, 16, {}), (2, 21, 8, 17, dict(estimator="picard")),
    (2, 16, [2, 5], 33, dict(n_intervals=2, schedule="sweeps")), (2, 17, 3, 40, dict(src="poly", ic="nodal", ic_data=np.zeros((1, 289)))),
    (5, 3, 3, 17, {}), (5, 4, 1, 16, {}), (5, 8, 1, 3, {})])
def test_tables_of_half_parts(dim, n, deg, nstar, kw):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] slab split", dim, n, deg, nstar, kw, flush=True)
    kw = dict(dict(src="longtime"), **kw)
    wl = W.small(dim=dim, n=n, M_deg=deg, M=2, T=0.4, f="sin", precision="fp32", nstar=nstar, **kw)
    rng = np.random.default_rng(n)
    if kw["src"] == "poly":
        wl = wl.with_(src_coeffs=0.1 * rng.standard_normal((n + 2) ** dim * (deg + 1)))
    U = [0.4 * rng.standard_normal((1, wl.nsp, d + 1)) for d in wl.degree]
    eps = []
    for mma in (1, 0):
        with H.Plan(wl) as plan:
            plan.hpsmc_set_option("sample_mfma", mma)
            plan.hpsmc_set_launch(1, 4, 2, 64)   # the matrix-core kernels take one path per lane
            assert plan.hpsmc_get_option("sample_mfma_active") == mma * (2 if dim == 5 else 1)
            for iv, u in enumerate(U):
                plan.hpsmc_set_nodes(iv, u)
            plan.hpsmc_sweep(3) if len(U) > 1 else plan.hpsmc_iterate(0, 3)
            eps.append(np.concatenate([plan.hpsmc_get_increment(iv)[0][0] for iv in range(len(U))]))
    assert np.max(np.abs(eps[0] - eps[1])) <= 1e-4 * (1.0 + np.max(np.abs(eps[1])))
