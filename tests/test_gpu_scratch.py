"""Plans whose device memory runs out at the scratch of the faster paths: creation
succeeds, the rounds run the kernel that needs none, and the results are those of the
full plan within the bounds of the parity tests.  Each of a plan's allocations is
refused in turn through the allocator hook; what a plan cannot do without is still
refused with HPSMC_ENOMEM."""
import numpy as np
import pytest

from paper_2608_22190_amd import workloads as W

pytestmark = pytest.mark.gpu


class _Hook:
    def __init__(self, refuse):
        import torch
        self.refuse, self.calls, self.sizes, self.torch = refuse, 0, [], torch

    def alloc(self, nbytes, stream):
        i = self.calls
        self.calls += 1
        self.sizes.append(nbytes)
        return 0 if i == self.refuse else self.torch.cuda.caching_allocator_alloc(nbytes)

    def free(self, ptr, stream):
        self.torch.cuda.caching_allocator_delete(ptr)


def _create(H, wl, refuse):
    hook = _Hook(refuse)
    H.hpsmc_set_allocator(hook.alloc, hook.free)
    try:
        return H.Plan(wl), hook
    except H.HpsmcError as e:
        assert e.status == -3   # ENOMEM
        return None, hook
    finally:
        H.hpsmc_set_allocator()


def _iterate(plan, U):
    plan.hpsmc_set_launch(1, 4, 2, 64)
    plan.hpsmc_set_nodes(0, U)
    plan.hpsmc_iterate(0, 1)
    forms = [plan.hpsmc_get_option(k) for k in ("sample_mfma_active", "sample_1d_active", "sample_1d_lattice_active")]
    return plan.hpsmc_get_nodes(0), plan.hpsmc_stats()["path_steps"], forms


@pytest.mark.parametrize("dim,n,M,prec,forms,optional,tol", [
    (1, 12, 300, "fp64", [0, 1, 1], [[0, 1, 0], [0, 1, 0]], 1e-12),       # descriptors, table -> windowed kernel
    (1, 18, 65, "fp64", [0, 1, 1], [[0, 1, 0], [0, 1, 0]], 1e-12),
    (2, 16, 20, "fp32", [1, 0, 0], [[0, 0, 0], [1, 0, 0]], 1e-4),         # images -> vector units; whole rounds
    (2, 6, 20, "fp64", [0, 0, 0], [[0, 0, 0]], 1e-12),                    # whole rounds
    (5, 2, 20, "fp32", [2, 0, 0], [[0, 0, 0], [2, 0, 0]], 1e-4)])
def test_a_refused_allocation_falls_back(dim, n, M, prec, forms, optional, tol):
    from paper_2608_22190_amd import hpsmc as H
    print("[case] scratch", dim, n, prec, flush=True)
    wl = W.small(dim=dim, n=n, M_deg=2, M=M, T=0.4, f="sin", src="longtime", nstar=120, precision=prec)
    U = np.random.default_rng(n).standard_normal((1, wl.nsp, 3)) * 0.4
    plan, hook = _create(H, wl, -1)
    with plan:
        ref, steps, got = _iterate(plan, U)
    assert got == forms
    seen = []
    for i in range(hook.calls):
        plan, h = _create(H, wl, i)
        if plan is None:
            assert not seen   # what may be missing comes last
            continue
        with plan:
            val, s, form = _iterate(plan, U)
        seen.append(form)
        assert s == steps
        assert np.max(np.abs(val - ref)) <= tol * (1.0 + np.max(np.abs(ref)))
    assert seen == optional


def test_a_gradient_after_one_that_ran_out_of_memory():
    from paper_2608_22190_amd import hpsmc as H
    print("[case] scratch gradient", flush=True)
    wl = W.small(dim=2, n=6, M_deg=2, M=20, iters=2, T=0.4, f="sin", src="longtime", nstar=60, precision="fp32", ic="phi",
                 ic_data=W.c5_coefficients(2, n=6).reshape(2, -1), n_instances=2)
    target = 0.1 * np.random.default_rng(0).standard_normal((2, wl.nsp))
    with H.Plan(wl) as plan:
        loss, grad = plan.hpsmc_loss_grad_c0(target)
    plan, hook = _create(H, wl, -1)
    failed = 0
    with plan:
        while failed < 20:
            hook.refuse = hook.calls + 1   # every call gets one buffer more and is refused the next
            try:
                again = plan.hpsmc_loss_grad_c0(target)
                break
            except H.HpsmcError as e:
                assert e.status == -3   # ENOMEM
                failed += 1
    assert failed == 8   # nine buffers
    assert np.array_equal(again[0], loss)
    assert np.max(np.abs(again[1] - grad)) <= 1e-5 * np.max(np.abs(grad))   # FP32 sums by atomics
