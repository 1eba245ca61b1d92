"""Off-node values of u* and v* against the oracle, for every rounding-up of the degree
(8, 16, 24, 32 time values in registers), one to four dimensions and point counts around
a block of 64.  Bound: each of the P + T terms that a value passes through per dimension
rounds at most as the nodal values themselves do, so 16 (P + T) times the change from
nodal values perturbed by one eps, the largest over the points."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu
CASES = [(1, 5, 1, 1), (1, 32, 7, 63), (1, 6, 8, 64), (2, 7, 15, 65), (2, 3, 16, 200), (1, 4, 23, 257), (2, 2, 24, 31),
         (1, 3, 31, 130), (3, 4, 3, 70), (3, 32, 1, 66), (4, 2, 2, 33), (4, 18, 1, 35)]


def _oracle(dim, n, deg, h, U, pts):
    Ut = O.reconstruct(dim, n, deg, U.reshape(-1))
    r = [O.evaluate(dim, n, deg, h, Ut, p[:dim], 2 * p[dim] / h - 1) for p in pts]
    return np.array([(u, lap - ut) for u, ut, lap in r])


@pytest.mark.parametrize("dim,n,deg,npts", CASES)
def test_eval_matches_the_oracle(dim, n, deg, npts):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] eval", dim, n, deg, npts, flush=True)
    h = 0.7
    wl = W.small(dim=dim, n=n, M_deg=deg, M=1, T=h, nstar=1, iters=1)
    rng = np.random.default_rng(n + deg)
    U = rng.standard_normal((1, wl.nsp, deg + 1)) * 0.4
    pts = np.concatenate([rng.uniform(-1, 1, (npts, dim)), rng.uniform(0, h, (npts, 1))], axis=1)
    with H.Plan(wl) as plan:
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_iterate(0, 0)   # reconstructs from U
        got = plan.hpsmc_eval(0, 0, pts)
    ref = _oracle(dim, n, deg, h, U, pts)
    moved = _oracle(dim, n, deg, h, U * (1 + np.finfo(float).eps * rng.choice([-1.0, 1.0], U.shape)), pts)
    bound = 16 * (n + 2 + deg + 1) * np.max(np.abs(moved - ref), axis=0)
    assert np.all(np.abs(got - ref) <= bound)
