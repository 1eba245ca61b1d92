"""Rounds of few batches, split into shares of steps over several blocks: the
increments against the FP64 oracle on the same Philox words where a round has
one batch (16 shares), as many batches as leave two shares and one share, with
rounds that are no multiple of the shares and paths carried over; two runs give
the same bits.  FP64 bound: 1e-12 of the iterate, as in the other parity tests
(the shares only regroup a path's sum).  FP32 matrix-core forms against the
vector-unit kernel to the 1e-4 bound of their own parity tests."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


def _iterate(wl, U, launch, **opt):
    from paper_2608_22190_amd import hpsmc as H
    with H.Plan(wl) as plan:
        for k, v in opt.items():
            plan.hpsmc_set_option(k, v)
        plan.hpsmc_set_launch(*launch)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 3)
        eps, _ = plan.hpsmc_get_increment(0)
        first = plan.hpsmc_stats()["path_steps"]
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 3)
        again, _ = plan.hpsmc_get_increment(0)
    assert np.array_equal(eps, again)
    return eps[0], first


@pytest.mark.parametrize("dim,n,deg,M,nstar,launch,kw", [
    (1, 3, 1, 5, 70, (1, 1, 2, 20), dict(quad="ball")),
    (1, 4, 2, 300, 33, (1, 4, 1, 16), dict(estimator="picard")),
    (2, 3, 2, 30, 50, (2, 2, 2, 20), {}),
    (2, 3, 2, 4000, 24, (1, 4, 1, 16), {}),          # 2 x 141 batches: two shares
    (2, 2, 1, 16000, 30, (1, 4, 1, 20), {}),         # 250 batches: three; later rounds more
    (2, 3, 2, 4260, 24, (1, 4, 1, 16), {}),          # 300 batches: two shares, more items than the grid's 256 blocks
    (2, 3, 2, 2120, 21, (1, 4, 1, 20), {}),          # 150 batches: five shares
    (2, 3, 2, 850, 24, (2, 4, 1, 16), {}),           # 30 batches of 512: sixteen; then fewer batches
    (2, 3, 2, 1000, 29, (1, 4, 1, 16), dict(estimator="picard")),   # 72 batches: ten
    (2, 3, 1, 37, 45, (1, 4, 4, 16), dict(estimator="picard", quad="ball")),
    (3, 2, 2, 50, 40, (2, 4, 2, 20), {}),
    (3, 10, 1, 2, 24, (1, 4, 2, 20), {}),            # LDS-chunked slabs
    (4, 2, 1, 60, 21, (1, 2, 2, 16), {}),
    (5, 2, 1, 33, 20, (1, 4, 2, 16), {})])
def test_shares_match_the_oracle_fp64(dim, n, deg, M, nstar, launch, kw):
    print("[case] shares", dim, n, deg, M, nstar, launch, kw, flush=True)
    wl = W.small(dim=dim, n=n, M_deg=deg, M=M, T=0.4, f="sin", src="longtime", nstar=nstar, **kw)
    U = np.random.default_rng(dim + n).standard_normal((1, wl.nsp, deg + 1)) * 0.4
    eps, steps = _iterate(wl, U, launch, sample_1d=0)
    Uo, _, so = O.Problem(wl).iterate(U[0].reshape(-1), iter_tag=3)
    ref = (Uo.reshape(wl.nsp, deg + 1) - U[0])[:, 1:].T.reshape(-1)
    assert steps == so
    assert np.max(np.abs(eps - ref)) <= 1e-12 * max(1.0, np.max(np.abs(Uo)))


@pytest.mark.parametrize("dim,n,deg,M,launch,kw", [
    (2, 16, 2, 3, (1, 4, 3, 20), {}), (2, 5, 2, 40, (1, 4, 3, 64), {}), (2, 16, 2, 9, (1, 4, 3, 36), dict(estimator="picard")),
    (2, 16, 1, 17, (1, 2, 2, 20), dict(quad="ball")), (5, 3, 1, 2, (1, 4, 2, 16), {}), (5, 3, 1, 150, (1, 2, 1, 20), {})])
def test_shares_of_the_matrix_core_kernels(dim, n, deg, M, launch, kw):
    print("[case] shares mma", dim, n, deg, M, launch, kw, flush=True)
    wl = W.small(dim=dim, n=n, M_deg=deg, M=M, T=0.4, f="sin", src="longtime", precision="fp32", nstar=150, **kw)
    U = np.random.default_rng(n).standard_normal((1, wl.nsp, deg + 1)) * 0.4
    em, sm = _iterate(wl, U, launch, sample_mfma=1)
    ev, sv = _iterate(wl, U, launch, sample_mfma=0)
    assert sm == sv
    assert np.max(np.abs(em - ev)) <= 1e-4 * (1.0 + np.max(np.abs(ev)))
