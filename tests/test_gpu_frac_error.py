"""Error against 64 bits of the fractional kernel's FP32 basis recurrence.

In the Picard form with f = u and nothing to add at the end, a path of one step
(N* = 1) that stays inside adds Delta w(x) sum_k U_k P_k(x) at its own node.  At 32
modes that is mostly the error of the recurrence P_{k+1} = (A_k x) P_k - C_k P_{k-1}
(A (x P) is up to twice as far off on such grids).  The bar is the same
sum in FP32, every product and sum rounded, with the weight rounded from 64 bits;
2% for the scatter of an rms and the weight's own last bit."""
import numpy as np
import pytest

import oracle as O
from paper_2608_22190_amd import workloads as W

F = np.float32


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(F)


def _recurrence(K, a):
    A, C = [a + 1.0], [0.0]
    for k in range(1, K):
        d = 2 * (k + 1) * (k + 2 * a + 1) * (2 * k + 2 * a)
        A.append((2 * k + 2 * a + 1) * (2 * k + 2 * a + 2) * (2 * k + 2 * a) / d)
        C.append(2 * (k + a) ** 2 * (2 * k + 2 * a + 2) / d)
    return A, C


def _sums(c, x, a):
    """(64-bit, FP32) sums over k of c[i][k] P_k(x)."""
    K = c.shape[1]
    A, C = _recurrence(K, a)
    xd = x.astype(np.float64)
    pm, pc, qm, qc = np.zeros_like(xd), np.ones_like(xd), np.zeros_like(x), np.ones_like(x)
    ref, s, c32 = 0.0, np.zeros((len(c), len(x)), F), c.astype(F)
    for k in range(K):
        ref = ref + c[:, k, None] * pc
        s = _fma(c32[:, k, None], qc[None], s)
        pm, pc = pc, A[k] * xd * pc - C[k] * pm
        qm, qc = qc, _fma(F(A[k]) * x, qc, -(F(C[k]) * qm))
    return ref, s


def _rms(e):
    return float(np.sqrt(np.mean(np.square(e))))


@pytest.mark.gpu
@pytest.mark.parametrize("alpha", [0.4, 1.0, 1.6])
def test_basis_recurrence_fp32(alpha):
    from paper_2608_22190_amd import hpsmc as H
    n, deg, inst, T = 32, 1, 300, 1e-4
    print("[case] frac error", alpha, flush=True)
    wl = W.small(dim=1, n=n, M_deg=deg, M=1, T=T, f="affine", f_param=[1.0, 0.0, 0, 0], src="none", ic="nodal",
                 ic_data=np.zeros((inst, n)), alpha=alpha, precision="fp32", estimator="picard", nstar=1, n_instances=inst)
    rng = np.random.default_rng(3)
    with H.Plan(wl) as plan:
        plan.hpsmc_set_launch(1, 4, 4, 64)
        x, t = plan.hpsmc_grid(0)
        U = np.zeros((inst, n, 2))
        # nodal values at the end time with independent coefficients in the scaled Jacobi basis
        P = np.array([_sums(np.eye(n), x.astype(F), 0.5 * alpha)[0]])[0]
        scale = np.sqrt(np.mean(P ** 2, axis=1))
        U[:, :, 1] = (1 - x * x) ** (0.5 * alpha) * ((rng.standard_normal((inst, n)) / scale) @ P)
        plan.hpsmc_set_nodes(0, U)
        plan.hpsmc_set_probe(1)
        plan.hpsmc_iterate(0, 1)
        got = plan.hpsmc_get_probe(0)[..., 0]
    c = np.array([O.frac_reconstruct(alpha, n, deg, u.reshape(-1)).reshape(n, 2).sum(axis=1) for u in U])
    xf = x.astype(F)
    ref, mod = _sums(c, xf, 0.5 * alpha)
    w, dl = (1 - xf.astype(np.float64) ** 2) ** (0.5 * alpha), np.float64(F(t[1] - t[0]))
    stays = got != 0.0
    assert stays.mean() > 0.5
    mod = (F(dl) * (w.astype(F) * mod)).astype(np.float64) / dl
    ker, bar = (got / dl - w * ref)[stays], (mod - w * ref)[stays]
    print(f"rms error {_rms(ker):.3e}, of the FP32 recurrence {_rms(bar):.3e}, {ker.size} values")
    assert _rms(ker) <= 1.02 * _rms(bar)

