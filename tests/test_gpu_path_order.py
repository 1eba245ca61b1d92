"""A path's value does not depend on what runs beside it: the same instance alone
(its few batches split into shares of steps over several blocks), among as many
others as leave fewer shares, and among so many that nothing is split gives the same
bits, path by path, as do its increments, and so do blocks of one wave and rounds of
another length.  Every round kernel that splits
rounds, both precisions, one and more paths a lane, the Picard and ball-point forms,
paths carried over rounds and rounds that are no multiple of the shares."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(wl, U, launch, opts):
    from paper_2608_22190_amd import hpsmc as H
    with H.Plan(wl) as plan:
        for k, v in opts.items():
            plan.hpsmc_set_option(k, v)
        plan.hpsmc_set_launch(*launch)
        plan.hpsmc_set_probe(min(wl.M, 8))
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 2)
        return plan.hpsmc_get_probe(0)[0], plan.hpsmc_get_increment(0)[0][0], plan.hpsmc_get_option("sample_mfma_active")


@pytest.mark.parametrize("dim,n,deg,M,nstar,launch,prec,mma,opts,kw", [
    (1, 4, 1, 30, 70, (1, 1, 2, 20), "fp64", 0, dict(sample_1d=0), {}),
    (1, 4, 1, 30, 70, (1, 2, 2, 20), "fp32", 0, {}, dict(quad="ball")),
    (2, 4, 1, 12, 150, (2, 2, 2, 64), "fp64", 0, {}, {}),
    (2, 4, 1, 12, 90, (1, 4, 2, 36), "fp64", 0, {}, dict(estimator="picard")),
    (2, 4, 1, 12, 90, (2, 4, 2, 36), "fp32", 0, {}, {}),
    (2, 4, 1, 12, 90, (4, 4, 2, 36), "fp32", 0, {}, {}),
    (2, 4, 1, 12, 90, (1, 4, 2, 36), "fp32", 1, {}, {}),
    (2, 16, 1, 3, 90, (1, 4, 3, 36), "fp32", 1, {}, {}),
    (2, 16, 1, 3, 90, (1, 4, 3, 36), "fp32", 1, {}, dict(estimator="picard")),
    (2, 16, 1, 3, 90, (1, 4, 3, 36), "fp32", 1, {}, dict(quad="ball")),
    (3, 3, 1, 7, 60, (2, 4, 2, 20), "fp32", 0, {}, {}),
    (5, 2, 1, 6, 60, (1, 4, 2, 20), "fp32", 2, dict(sample_split=0), {})])
def test_path_values_do_not_depend_on_their_company(dim, n, deg, M, nstar, launch, prec, mma, opts, kw):
    print("[case] path order", dim, n, M, launch, prec, kw, flush=True)
    rng = np.random.default_rng(n)
    U = rng.standard_normal((1, n ** dim, deg + 1)) * 0.4
    runs = []
    for inst, shape in ((1, launch), (60, launch), (800, launch), (1, (launch[0], 1, 3, 52))):
        wl = W.small(dim=dim, n=n, M_deg=deg, M=M, T=0.3, f="sin", src="longtime", precision=prec, nstar=nstar,
                     n_instances=inst, **kw)
        p, e, active = _run(wl, np.repeat(U, inst, axis=0), shape, opts)
        assert active == mma
        runs.append((p, e))
    assert np.any(runs[0][0] != 0.0)
    for p, e in runs[1:]:
        assert np.array_equal(p, runs[0][0])
        assert np.array_equal(e, runs[0][1])
