"""The slab adjoint with its chunks of 32 steps split into shares over several blocks:
one share, two, the cap of 64, shares that start and end inside a group, groups of
unequal step counts (shares past an instance's last chunk).  FP64 gradients against the
oracle's reverse mode to the 1e-10 of the other adjoint tests: the shares only regroup
the sums."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,nstar,I", [
    (1, 3, [480], 1), (1, 3, [513], 1), (2, 2, [333, 701], 2), (1, 2, [40, 3, 4000], 3), (2, 3, [9000, 12000], 1)])
def test_shares_of_the_slab_adjoint(dim, n, nstar, I):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] adjoint shares", dim, n, nstar, I, flush=True)
    rng = np.random.default_rng(n)
    c0 = rng.standard_normal((I, n ** dim)) / (1.0 + np.arange(n ** dim))
    wl = W.small(dim=dim, n=n, M_deg=len(nstar), M=5, T=0.5, iters=2, f="sin", f_param=[0.7, 0.1, 0, 0], src="longtime",
                 ic="phi", ic_data=c0, n_instances=I).with_(nstar=nstar, nstar_mode="array")
    target = rng.standard_normal((I, wl.nsp))
    with H.Plan(wl) as plan:
        loss, grad = plan.hpsmc_loss_grad_c0(target)
    pb = O.Problem(wl)
    for i in range(I):
        lo, go = pb.loss_grad(c0[i], target[i], inst=i)
        assert abs(loss[i] - lo) <= 1e-11 * (1 + abs(lo))
        assert np.max(np.abs(grad[i] - go)) <= 1e-10 * (1 + np.max(np.abs(go)))
