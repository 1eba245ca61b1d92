"""The work a user of this library has it do, as cases that can be timed and checked.

A case is a dict of plain values.  ``prepare`` builds the plan and the inputs a
program holds before the call, ``run`` makes one pass through the public entry
points of the binding, ``work`` counts what the pass cannot do without, and
``exact`` evaluates the same estimator in 64 bits with torch and NumPy alone.

Kinds of pass:
  step      one residual iteration of interval 0 from given nodal values
            (hpsmc_set_nodes, hpsmc_iterate, hpsmc_get_nodes, hpsmc_get_increment)
  solve     a whole solve of every interval from given initial nodal values
  sweep     one Jacobi-in-time sweep over all intervals from given nodal values
  gradient  terminal misfit and its gradient through the autograd function
  evaluate  the reconstruction at arbitrary points, host arrays in and out

Results of plans that sample in FP32 are handed on as float32: they hold no
more digits than that.
"""
import math

import numpy as np
import torch

from paper_2608_22190_amd import hpsmc
from paper_2608_22190_amd.workloads import Workload, c5_coefficients

DEFAULTS = dict(kind="step", dim=1, n=8, deg=6, T=0.5, M=64, iters=1, prec="fp64", f="u_minus_u3", src="sin_decay",
                est="residual", quad="centre", intervals=1, mesh="uniform", inst=1, alpha=2.0, npts=0, launch="",
                graph=False)


def listed():
    return [
        # the smallest call: one iteration of a coarse line problem inside a user's own
        # loop; launches and latency are all there is
        dict(name="line_step", kind="step", dim=1, n=6, deg=4, T=0.5, M=64),
        # the single-step accuracy experiment on a line: 16 x 16 nodes, FP64, a
        # whole solve replayed as a graph
        dict(name="line_solve", kind="solve", dim=1, n=16, deg=16, T=1.0, M=4096, iters=5, graph=True,
             launch="1,4,4,512"),
        # an ordinary small plane problem with the library's default launch shape:
        # odd mode count, a sample count that fills no wave, FP32 sampling
        dict(name="plane_solve", kind="solve", dim=2, n=9, deg=5, T=0.5, M=200, iters=3, prec="fp32", f="sin",
             src="longtime"),
        # the long-time experiment: 24 x 24 x 16 nodes of a unit interval, FP32
        # sampling, a slice of the samples (the benchmark's workload)
        dict(name="plane_step", kind="step", dim=2, n=24, deg=16, T=1.0, M=256, prec="fp32", f="sin", src="longtime",
             launch="1,4,3,256"),
        # the same grid sampled in FP64 (a quarter of the interval), what the final
        # iterations of a solve to tolerance run
        dict(name="plane_step_fp64", kind="step", dim=2, n=24, deg=16, T=0.25, M=128, f="sin", src="longtime",
             launch="2,4,2,256"),
        # the initial-layer experiment: twelve geometric intervals of growing
        # degree swept together
        dict(name="plane_sweep", kind="sweep", dim=2, n=20, deg=26, T=1.0, M=64, prec="fp32", f="u2_over_1pu2",
             src="none", intervals=12, mesh="geometric", launch="1,4,3,256"),
        # the classical Monte Carlo (Picard) form on the long-time interval
        dict(name="plane_picard", kind="step", dim=2, n=24, deg=16, T=1.0, M=64, prec="fp32", f="sin", src="longtime",
             est="picard", launch="1,4,3,512"),
        # a three-dimensional iteration, FP32, default launch shape
        dict(name="solid_step", kind="step", dim=3, n=8, deg=6, T=0.5, M=64, prec="fp32", f="u_minus_u3",
             src="cos_decay"),
        # the five-dimensional experiment: 8^5 x 8 nodes, a slice of the samples
        dict(name="five_dim_step", kind="step", dim=5, n=8, deg=8, T=1.0, M=2, prec="fp32", f="neg_u3",
             src="cos_decay", launch="1,4,2,16"),
        # batched gradients with respect to the initial data (forward and adjoint)
        dict(name="gradient", kind="gradient", dim=2, n=16, deg=12, T=0.5, M=16, iters=2, prec="fp32", f="sin",
             src="longtime", inst=8, launch="1,4,3,256"),
        # the fractional long-time experiment: eight intervals, replayed as a graph
        dict(name="frac_solve", kind="solve", dim=1, n=11, deg=6, T=4.0, M=8192, iters=6, prec="fp32",
             src="frac_longtime", intervals=8, alpha=0.4, graph=True, launch="1,4,4,128"),
        # off-node values of a plane solution for output and comparison
        dict(name="evaluate", kind="evaluate", dim=2, n=16, deg=12, T=0.5, M=4, f="sin", src="longtime", npts=20000),
    ]


# families of draw(): the ranges of the listed cases
_FAMILIES = (
    dict(kind="step", dim=1, n=(4, 24), deg=(2, 16), T=(0.1, 1.0), M=(16, 4096)),
    dict(kind="solve", dim=1, n=(4, 20), deg=(2, 16), T=(0.1, 1.0), M=(64, 8192), iters=(2, 5), graph=True,
         launch="1,4,4,512"),
    dict(kind="step", dim=1, n=(4, 16), deg=(2, 10), T=(0.1, 1.0), M=(64, 2048), est="picard"),
    dict(kind="solve", dim=2, n=(4, 12), deg=(2, 8), T=(0.1, 0.5), M=(16, 1024), iters=(2, 4), prec="fp32", f="sin",
         src="longtime"),
    dict(kind="step", dim=2, n=(12, 26), deg=(4, 16), T=(0.1, 1.0), M=(16, 256), prec="fp32", f="sin", src="longtime",
         launch="1,4,3,256"),
    dict(kind="step", dim=2, n=(6, 24), deg=(4, 16), T=(0.1, 1.0), M=(8, 128), f="sin", src="longtime",
         launch="2,4,2,256"),
    dict(kind="step", dim=2, n=(8, 24), deg=(4, 12), T=(0.1, 0.5), M=(16, 128), prec="fp32", f="sin", src="longtime",
         est="picard", launch="1,4,3,512"),
    dict(kind="step", dim=2, n=(8, 24), deg=(4, 12), T=(0.1, 0.5), M=(16, 128), prec="fp32", f="sin", src="longtime",
         quad="ball", launch="1,4,3,256"),
    dict(kind="sweep", dim=2, n=(6, 20), deg=(8, 26), T=(0.2, 1.0), M=(16, 128), prec="fp32", f="u2_over_1pu2",
         src="none", mesh="geometric", intervals=(3, 12), launch="1,4,3,256"),
    dict(kind="step", dim=3, n=(3, 12), deg=(2, 8), T=(0.1, 0.5), M=(8, 256), prec="fp32", src="cos_decay"),
    dict(kind="step", dim=3, n=(3, 10), deg=(2, 6), T=(0.1, 0.5), M=(8, 128), src="cos_decay"),
    dict(kind="step", dim=5, n=(3, 8), deg=(2, 8), T=(0.1, 1.0), M=(1, 64), prec="fp32", f="neg_u3", src="cos_decay",
         launch="1,4,2,16"),
    dict(kind="gradient", dim=2, n=(6, 18), deg=(3, 12), T=(0.1, 0.5), M=(8, 64), iters=(1, 3), prec="fp32", f="sin",
         src="longtime", inst=(1, 8), launch="1,4,3,256"),
    dict(kind="solve", dim=1, n=(6, 16), deg=(3, 8), T=(1.0, 8.0), M=(512, 8192), iters=(2, 6), prec="fp32",
         src="frac_longtime", intervals=(2, 8), alpha=(0.4, 1.6), graph=True, launch="1,4,4,128"),
    dict(kind="solve", dim=1, n=(6, 12), deg=(3, 6), T=(1.0, 4.0), M=(512, 8192), iters=(2, 4), src="frac_longtime",
         intervals=(2, 6), alpha=(0.4, 1.6), graph=True, launch="1,4,3,512"),
    dict(kind="evaluate", dim=2, n=(6, 24), deg=(4, 16), T=(0.1, 1.0), M=4, f="sin", src="longtime", npts=(100, 40000)),
)


def draw(rng):
    """One more case of the ranges above, its samples scaled down until it costs no
    more than the largest listed one."""
    fam = rng.choice(_FAMILIES)
    c = {}
    for k, v in fam.items():
        if not isinstance(v, tuple):
            c[k] = v
        elif isinstance(v[0], float):
            c[k] = round(math.exp(rng.uniform(math.log(v[0]), math.log(v[1]))), 3)
        elif v[1] > 10 * v[0]:
            c[k] = int(round(math.exp(rng.uniform(math.log(v[0]), math.log(v[1])))))
        else:
            c[k] = rng.randint(*v)
    if c["kind"] == "gradient":
        c["n"] = min(c["n"], 18)
    # bytes and flops at the rates such passes reach, and the walk's longest path,
    # one step after another
    rate = {1: 8e12, 2: 5e13 if c.get("prec") == "fp32" else 2e13, 3: 1e13, 5: 6e13}[c["dim"]]
    while c["M"] > 1 and c["kind"] != "evaluate" and work(c)["flops"] / rate > 0.25:
        c["M"] = max(1, c["M"] * 3 // 4)
    while c["kind"] not in ("evaluate",) and _longest(c) * 2e-6 > 0.25 and c["T"] > 0.02:
        c["T"] = round(c["T"] * 0.7, 4)
    return c


def _full(case):
    return {**DEFAULTS, **{k: v for k, v in case.items() if k != "name"}}


def _workload(c, seed=0):
    if c["mesh"] == "geometric":
        tb = [0.0] + [c["T"] * 0.2 ** (c["intervals"] - k) for k in range(1, c["intervals"] + 1)]
        top = c["deg"]
        deg = [max(2, top - 2 * (c["intervals"] - k)) for k in range(1, c["intervals"] + 1)]
    else:
        tb = [c["T"] * k / c["intervals"] for k in range(c["intervals"] + 1)]
        deg = [c["deg"]] * c["intervals"]
    kw = {}
    if c["kind"] == "gradient":
        kw = dict(ic="phi", ic_data=c5_coefficients(c["inst"], n=c["n"], seed=seed).reshape(c["inst"], -1))
    elif c["src"] == "none":
        kw = dict(ic="singular", ic_param=[0.5, 0.0, 0.0, 0.0])
    return Workload(name="case", dim=c["dim"], n=c["n"], t_breaks=tb, degree=deg, f=c["f"], src=c["src"], M=c["M"],
                    iters=c["iters"], seed=seed, schedule="sweeps" if c["kind"] == "sweep" else "sequential",
                    n_instances=c["inst"], precision=c["prec"], estimator=c["est"], quad=c["quad"], alpha=c["alpha"], **kw)


def _rng(c, seed):
    return np.random.default_rng(977 * int(seed) + c["n"])


def _initial(c, seed, x):
    """Smooth initial nodal values [n^d], zero on the boundary, made from the seed."""
    r, g = _rng(c, seed), np.ones(1)
    for _ in range(c["dim"]):
        a = r.uniform(-0.4, 0.4, 3)
        w = (1 - x * x) ** (0.5 * c["alpha"] if c["alpha"] < 2 else 1.0)
        g = np.multiply.outer(g, w * (1 + a[0] * x + a[1] * x * x + a[2] * np.sin(2 * x)))
    return 0.8 * g.reshape(-1)


def _nodal(c, seed, x, t, iv):
    """Nodal values [1][n^d][M+1] of an iterate: smooth in space and time."""
    u0 = _initial(c, seed, x)
    a = _rng(c, seed + 31 * iv + 7).uniform(-0.5, 0.5, 2)
    return (u0[:, None] * (np.exp(-t) * (1 + a[0] * t + a[1] * t * t))[None, :])[None]


def prepare(case, seed):
    c = _full(case)
    wl = _workload(c, seed)
    plan = hpsmc.Plan(wl)
    if c["launch"]:
        plan.hpsmc_set_launch(*(int(v) for v in c["launch"].split(",")))
    if c["graph"]:
        plan.hpsmc_set_option("graph", 1)
    s = dict(c=c, plan=plan, stream=torch.cuda.current_stream())
    grid = [plan.hpsmc_grid(iv) for iv in range(len(wl.degree))]
    dev = torch.device("cuda")
    if c["kind"] in ("step", "sweep", "evaluate"):
        s["U"] = [torch.from_numpy(_nodal(c, seed, x, t, iv)).to(dev) for iv, (x, t) in enumerate(grid)]
    if c["kind"] == "solve":
        plan.hpsmc_set_initial_nodes(_initial(c, seed, grid[0][0])[None])
    if c["kind"] == "gradient":
        s["c0"] = torch.from_numpy(wl.ic_data.copy()).to(dev)
        s["target"] = torch.from_numpy(0.1 * _rng(c, seed).standard_normal((c["inst"], c["n"] ** c["dim"]))).to(dev)
        s["loss"] = hpsmc.smc_loss_function()
    if c["kind"] == "evaluate":
        plan.hpsmc_set_nodes(0, s["U"][0])
        plan.hpsmc_iterate(0, 0)
        r = _rng(c, seed + 1)
        s["pts"] = np.concatenate([r.uniform(-1, 1, (c["npts"], c["dim"])), r.uniform(0, c["T"], (c["npts"], 1))], 1)
    s["out"] = [torch.empty((c["inst"], c["n"] ** c["dim"], m + 1), dtype=torch.float64, device=dev) for m in wl.degree]
    torch.cuda.synchronize()
    return s


def _handed_on(c, v):
    if c["prec"] != "fp32":
        return v
    return v.to(torch.float32) if isinstance(v, torch.Tensor) else v.astype(np.float32)


def run(s):
    c, plan, stream = s["c"], s["plan"], s["stream"]
    kind = c["kind"]
    if kind == "step":
        plan.hpsmc_set_nodes(0, s["U"][0], stream=stream)
        plan.hpsmc_iterate(0, 0, stream=stream)
        U = plan.hpsmc_get_nodes(0, out=s["out"][0], stream=stream)
        eps, ssq = plan.hpsmc_get_increment(0, stream=stream)
        return {k: _handed_on(c, v) for k, v in (("U", U), ("eps", eps), ("sumsq", ssq))}
    if kind == "solve":
        plan.hpsmc_solve(stream=stream)
    elif kind == "sweep":
        for iv, U in enumerate(s["U"]):
            plan.hpsmc_set_nodes(iv, U, stream=stream)
        plan.hpsmc_sweep(0, stream=stream)
    elif kind == "gradient":
        c0 = s["c0"].detach().requires_grad_(True)
        loss = s["loss"].apply(c0, plan, s["target"], stream)
        loss.sum().backward()
        return {"loss": _handed_on(c, loss.detach()), "grad": _handed_on(c, c0.grad)}
    else:
        return plan.hpsmc_eval(0, 0, s["pts"], stream=stream)
    return [_handed_on(c, plan.hpsmc_get_nodes(iv, out=o, stream=stream)) for iv, o in enumerate(s["out"])]


# ---------------------------------------------------------------- work
def _grid_x(c):
    """Spatial nodes: Gauss-Jacobi (1,1), or (alpha/2, alpha/2) for the fractional operator."""
    a = 0.5 * c["alpha"] if c["alpha"] < 2 else 1.0
    k = np.arange(1, c["n"], dtype=np.float64)
    e = np.sqrt(_beta(k, a))
    return np.linalg.eigvalsh(np.diag(e, 1) + np.diag(e, -1))


def _beta(k, a):
    return k * (k + 2 * a) / ((2 * k + 2 * a + 1) * (2 * k + 2 * a - 1))


def _grid_xi(M):
    """Lobatto nodes on [-1, 1]: the end points and the zeros of L'_M = Gauss-Jacobi (1,1)."""
    k = np.arange(1, M - 1, dtype=np.float64)
    e = np.sqrt(_beta(k, 1.0))
    mid = np.linalg.eigvalsh(np.diag(e, 1) + np.diag(e, -1)) if M > 1 else np.zeros(0)
    return np.concatenate([[-1.0], mid, [1.0]])


def _survival(x, s):
    """Probability that a one-dimensional walk of generator d^2/dx^2 from x is inside after time s."""
    k = np.arange(60)[:, None, None]
    m = (2 * k + 1) * math.pi / 2
    p = (4 / math.pi) * (-1.0) ** k / (2 * k + 1) * np.cos(m * x[None, :, None]) * np.exp(-m * m * s[None, None, :])
    return np.clip(p.sum(0), 0.0, 1.0)


def _evaluations(c):
    """Expected residual evaluations of one iteration over all intervals."""
    wl = _workload(c)
    ns, _ = hpsmc.resolve_nstar(wl)
    x, total, o = _grid_x(c), 0.0, 0
    for iv, m in enumerate(wl.degree):
        h = wl.t_breaks[iv + 1] - wl.t_breaks[iv]
        for xi, N in zip(_grid_xi(m)[1:], ns[o:o + m]):
            span = 0.5 * (xi + 1) * h
            if c["alpha"] < 2:
                total += 0.6 * N
                continue
            g = (np.arange(200) + 0.5) / 200
            g, w = span * g ** 2, span * 2 * g / 200   # finer where the boundary nodes leave
            total += N / span * float((_survival(x, g).mean(0) ** c["dim"] * w).sum())
        o += m
    return total * c["n"] ** c["dim"] * c["M"] * c["inst"]


def _longest(c):
    """Walk steps one after another in a pass."""
    c = _full(c)
    return int(hpsmc.resolve_nstar(_workload(c))[0].max()) * c["iters"] * c["intervals"] ** (c["kind"] == "solve")


def work(case):
    """Flops: the two contractions of u* and v* with the tensor basis at every residual
    evaluation (the misfit's gradient contracts twice).  Bytes: the nodal values and
    results in and out."""
    c = _full(case)
    wl = _workload(c)
    nodes = 8 * c["inst"] * c["n"] ** c["dim"] * sum(m + 1 for m in wl.degree)
    P, d = c["n"] + (2 if c["alpha"] >= 2 else 0), c["dim"]
    per = (2 if c["est"] == "picard" else 4) * sum(P ** (k + 1) for k in range(d)) + 3 * d * P
    if c["kind"] == "evaluate":
        T1 = c["deg"] + 1
        return {"bytes": 8 * c["npts"] * (d + 3) + nodes, "flops": 4.0 * c["npts"] * P ** d + 2.0 * P ** d * T1 * (P * d + T1)}
    flops = per * _evaluations(c) * c["iters"] * (2 if c["kind"] == "gradient" else 1)
    return {"bytes": 4 * nodes if c["kind"] == "step" else 2 * nodes, "flops": flops}


# ---------------------------------------------------------------- 64-bit reference
def _leg(P, x):
    """Legendre values [..., P] of a float64 tensor."""
    L = [torch.ones_like(x), x]
    for k in range(1, P - 1):
        L.append(((2 * k + 1) * x * L[k] - k * L[k - 1]) / (k + 1))
    return torch.stack(L[:P], -1)


def _leg_d(P):
    """Derivative matrix in Legendre coefficients: (c')_i = sum_j D[i, j] c_j."""
    D = np.zeros((P, P))
    for j in range(P):
        for i in range(j - 1, -1, -2):
            D[i, j] = 2 * i + 1
    return D


def _jac(K, a, x):
    """Orthonormal-recurrence Jacobi values [..., K], parameters (a, a), p_0 = 1."""
    b = [0.0] + [math.sqrt(_beta(k, a)) for k in range(1, K + 1)]
    p = [torch.ones_like(x), x / b[1]]
    for k in range(1, K - 1):
        p.append((x * p[k] - b[k] * p[k - 1]) / b[k + 1])
    return torch.stack(p[:K], -1)


def _philox(c0, c1, c2, c3, k0, k1):
    m = 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & m) ^ c1 ^ k0, p1 & m, ((p0 >> 32) & m) ^ c3 ^ k1, p0 & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _f(kind, u):
    return {"u_minus_u3": lambda: u - u ** 3, "sin": lambda: torch.sin(u), "neg_u3": lambda: -u ** 3,
            "u2_over_1pu2": lambda: u * u / (1 + u * u)}[kind]()


class _Exact:
    """The estimator of one case in 64 bits: interpolation, walks and sums as the
    method states them, every path at once."""

    def __init__(self, c, seed):
        self.c, self.seed = c, int(seed)
        self.wl = _workload(c, seed)
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.x = _grid_x(c)
        ns, _ = hpsmc.resolve_nstar(self.wl)   # the path lengths are an input of the method
        o = np.cumsum([0] + list(self.wl.degree))
        self.ns = [ns[o[i]:o[i + 1]].astype(np.int64) for i in range(len(self.wl.degree))]
        self.frac = c["alpha"] < 2
        if self.frac:
            a, K = 0.5 * c["alpha"], 60
            k = np.arange(1, 160, dtype=np.float64)
            e = np.sqrt(_beta(k, a))
            ev, V = np.linalg.eigh(np.diag(e, 1) + np.diag(e, -1))
            J = _jac(K, a, torch.from_numpy(ev)).numpy()
            lam = np.array([math.exp(math.lgamma(p + c["alpha"] + 1) - math.lgamma(p + 1)) for p in range(K)])
            self.gk = self.t(lam * (J * (V[0] ** 2 * np.sin(ev))[:, None]).sum(0))
            self.lam = lam

    def t(self, v):
        return torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=self.dev)

    def uniform(self, w):
        return ((w >> 8).double() + 0.5) * 2.0 ** -24 if self.c["prec"] == "fp32" else (w.double() + 0.5) * 2.0 ** -32

    def start(self, U0, iv):
        return np.repeat(U0[:, None], self.wl.degree[iv] + 1, 1)

    def tables(self, U, iv):
        """Modal tensors of u* and v* [n^d modes..., M+1] (fractional: and of the operator)."""
        c, d, P, M = self.c, self.c["dim"], self.c["n"] + 2, self.wl.degree[iv]
        h = self.wl.t_breaks[iv + 1] - self.wl.t_breaks[iv]
        B = np.linalg.inv(_leg(M + 1, torch.from_numpy(_grid_xi(M))).numpy())
        x = torch.from_numpy(self.x)
        Dt = _leg_d(M + 1) * 2 / h
        if self.frac:
            a = 0.5 * c["alpha"]
            A = np.linalg.inv(_jac(c["n"], a, x).numpy() * ((1 - self.x ** 2) ** a)[:, None])
            C = A @ U @ B.T
            return self.t(np.stack([C, -(C @ Dt.T), self.lam[:c["n"], None] * C], 0))
        L = _leg(P, x).numpy()
        A = np.linalg.inv(L[:, :c["n"]] - L[:, 2:])   # phi_p = L_p - L_{p+2}: values to coefficients
        E = np.zeros((P, c["n"]))
        for p in range(c["n"]):
            E[p, p], E[p + 2, p] = 1.0, -1.0
        C = U.reshape((c["n"],) * d + (M + 1,))
        for i in range(d):
            C = np.moveaxis(np.tensordot(E @ A, C, (1, i)), 0, i)
        C = C @ B.T
        D2 = _leg_d(P) @ _leg_d(P)
        V = -(C @ Dt.T)
        for i in range(d):
            V = V + np.moveaxis(np.tensordot(D2, C, (1, i)), 0, i)
        return self.t(np.stack([C, V], 0))

    def source(self, X, t):
        c, d = self.c, self.c["dim"]
        if c["src"] == "none":
            return 0.0
        x = [X[..., i] for i in range(d)]
        if c["src"] in ("sin_decay", "cos_decay"):
            fn, lam = (torch.sin, math.pi ** 2) if c["src"] == "sin_decay" else (torch.cos, math.pi ** 2 / 4)
            u = torch.exp(-t)
            for v in x:
                u = u * fn(v * math.sqrt(lam))
            return -u + d * lam * u - _f(c["f"], u)
        Tt = torch.exp(torch.cos(t)) / (1 + t * t)
        Tp = Tt * (-torch.sin(t) - 2 * t / (1 + t * t))
        om, s = [1 - v * v for v in x], sum(x)
        a, S, Co = math.prod(om[1:], start=om[0]), torch.sin(s), torch.cos(s)
        rest = [math.prod([om[j] for j in range(d) if j != i], start=torch.ones_like(s)) for i in range(d)]
        lap = S * sum(-2 * r for r in rest) + 2 * Co * sum(-2 * v * r for v, r in zip(x, rest)) - d * a * S
        return a * S * Tp - lap * Tt - _f(c["f"], a * S * Tt)

    def jump(self, om):
        """R-free jump of the alpha-stable exit law: x^{-1/2}, I_x(a, 1-a) = om."""
        a = 0.5 * self.c["alpha"]
        one = torch.ones(1, dtype=torch.float64, device=self.dev)

        def series(p, x):   # I_x(p, 1-p) p B / (x^p (1-x)^(1-p))
            s, term = torch.ones_like(x), torch.ones_like(x)
            for k in range(60):
                term = term * x * ((k + 1) / (p + 1 + k))
                s = s + term
            return s
        lB = math.lgamma(a) + math.lgamma(1 - a)
        half = float(torch.exp(a * torch.log(one / 2) + (1 - a) * torch.log(one / 2) - lB - math.log(a)) * series(a, one / 2))
        low = om <= half
        p = torch.where(low, torch.full_like(om, a), torch.full_like(om, 1 - a))
        ly = torch.log(torch.where(low, om, 1 - om))
        z = torch.clamp((ly + lB + torch.log(p)) / p, max=-math.log(2))
        for _ in range(7):
            x = torch.exp(z)
            s = series(p, x)
            I = p * z + (1 - p) * torch.log1p(-x) - lB - torch.log(p) + torch.log(s)
            z = torch.clamp(z - (I - ly) * (1 - x) * s / p, max=-math.log(2))
        return torch.where(low, torch.exp(-0.5 * z), 1 / torch.sqrt(-torch.expm1(z) + (z == 0)))

    def estimate(self, U, iv, tag):
        """(eps [M][n^d], sum S^2) of one iteration from U [n^d][M+1]."""
        c, d, dev, n, M = self.c, self.c["dim"], self.dev, self.c["n"], self.wl.degree[iv]
        nsp, S = n ** d, c["M"]
        t0, h = self.wl.t_breaks[iv], self.wl.t_breaks[iv + 1] - self.wl.t_breaks[iv]
        tab = self.tables(U, iv)
        P = tab.shape[1]
        span_l = 0.5 * (_grid_xi(M)[1:] + 1) * h
        N_l = self.ns[iv]
        acc = torch.zeros(M * nsp * S, dtype=torch.float64, device=dev)
        idx = torch.arange(M * nsp * S, device=dev)
        l, j, smp = idx // (nsp * S), (idx // S) % nsp, idx % S
        grids = np.stack(np.meshgrid(*([self.x] * d), indexing="ij"), -1).reshape(nsp, d)
        X = self.t(grids)[j]
        dl_l = span_l / N_l
        if self.frac:
            R_l = (dl_l * math.gamma(1 + c["alpha"])) ** (1 / c["alpha"])
        else:
            R_l = np.sqrt(2 * d * dl_l)
        dl_t, R_t, sp_t, N_t = self.t(dl_l), self.t(R_l), self.t(span_l), torch.as_tensor(N_l, device=dev)
        k0, k1 = self.seed & 0xFFFFFFFF, (self.seed >> 32) & 0xFFFFFFFF
        c3 = (iv << 8) | tag
        words = None
        for q in range(int(N_l.max())):
            keep = N_t[l] > q
            if c["est"] == "picard" and not bool(keep.all()):   # paths that reached t_{n-1} inside
                done = ~keep
                acc[idx[done]] += self.evaluate(tab[:1], X[done], l[done], -torch.ones(M, dtype=torch.float64, device=dev))[0]
            if q % 16 == 0 or not bool(keep.all()):
                if not bool(keep.all()):
                    idx, l, j, smp, X = idx[keep], l[keep], j[keep], smp[keep], X[keep]
                    words = None if words is None else [w[keep] for w in words]
            if idx.numel() == 0:
                break
            node = j + nsp * l
            z = torch.full_like(node, c3)
            per = {1: 2 if self.frac else 128, 2: 4}.get(d, 1)
            if q % per == 0 or words is None:
                blk = q // per * (2 if d == 5 else 1)
                words = _philox(node, smp, torch.full_like(node, blk), z, k0, k1)
                if d == 5:
                    words = words + _philox(node, smp, torch.full_like(node, blk + 1), z, k0, k1)
            if self.frac:
                Jq = self.jump(self.uniform(words[2 * (q % 2)])) * R_t[l]
                dirs = torch.where((words[2 * (q % 2) + 1] & 1) == 1, 1.0, -1.0).double()[:, None]
            elif d == 1:
                Jq = R_t[l]
                dirs = torch.where((words[(q >> 5) & 3] >> (q & 31)) & 1 == 1, 1.0, -1.0).double()[:, None]
            elif d == 2:
                Jq = R_t[l]
                ang = 2 * math.pi * self.uniform(words[q & 3])
                dirs = torch.stack([torch.cos(ang), torch.sin(ang)], -1)
            else:
                Jq, g = R_t[l], []
                for k in range((d + 1) // 2):
                    r = torch.sqrt(-2 * torch.log(self.uniform(words[2 * k])))
                    ang = 2 * math.pi * self.uniform(words[2 * k + 1])
                    g += [r * torch.cos(ang), r * torch.sin(ang)]
                dirs = torch.stack(g[:d], -1)
                dirs = dirs / dirs.norm(dim=-1, keepdim=True)
            Y = X + Jq[:, None] * dirs
            inside = (Y.abs() < 1).all(-1)
            if not bool(inside.all()):
                idx, l, j, smp, X, Y = (v[inside] for v in (idx, l, j, smp, X, Y))
                words = [w[inside] for w in words]
            if idx.numel() == 0:
                break
            tau = sp_t - q * dl_t
            xi = 2 * tau / h - 1
            u, v = self.evaluate(tab, X, l, xi)[:2]
            t = (t0 + tau)[l]
            if self.frac:
                F = self.last
                w = (1 - X[:, 0] ** 2) ** (0.5 * c["alpha"])
                Tt = torch.exp(torch.cos(t)) / (1 + t * t)
                Tp = Tt * (-torch.sin(t) - 2 * t / (1 + t * t))
                g = torch.sin(X[:, 0])
                G = _jac(self.gk.numel(), 0.5 * c["alpha"], X[:, 0]) @ self.gk
                r = _f(c["f"], w * u) + w * g * Tp + G * Tt - _f(c["f"], w * g * Tt) + w * v - F
            else:
                r = _f(c["f"], u) + self.source(X, t) + (v if c["est"] == "residual" else 0.0)
            acc[idx] += dl_t[l] * r
            X = Y
        else:
            if c["est"] == "picard" and idx.numel():
                acc[idx] += self.evaluate(tab[:1], X, l, -torch.ones(M, dtype=torch.float64, device=dev))[0]
        S_ = acc.reshape(M, nsp, S)
        return S_.mean(-1).cpu().numpy(), (S_ * S_).sum(-1).cpu().numpy()

    def evaluate(self, tab, X, l, xi):
        """u, v (and the operator's series) at points X of node times l, whose reference times are xi."""
        d, P, K = self.c["dim"], tab.shape[1], tab.shape[0]
        slab = tab @ _leg(tab.shape[-1], xi).T.contiguous()       # [K][P..][M]
        slab = slab.movedim(-1, 0).reshape(xi.numel(), K, -1)
        outs = torch.empty(K, X.shape[0], dtype=torch.float64, device=X.device)
        lo = 0
        counts = torch.bincount(l, minlength=xi.numel()).tolist()
        basis = _jac if self.frac else None
        for m, cnt in enumerate(counts):   # the paths stay sorted by node time
            for b in range(lo, lo + cnt, 65536):
                e = min(lo + cnt, b + 65536)
                L = [basis(P, 0.5 * self.c["alpha"], X[b:e, i].contiguous()) if basis else _leg(P, X[b:e, i].contiguous())
                     for i in range(d)]
                split = (d + 1) // 2
                lead, tail = L[0], L[split] if split < d else None
                for i in range(1, split):
                    lead = (lead[:, :, None] * L[i][:, None, :]).reshape(e - b, -1)
                for i in range(split + 1, d):
                    tail = (tail[:, :, None] * L[i][:, None, :]).reshape(e - b, -1)
                for k in range(K):
                    s = slab[m, k]
                    outs[k, b:e] = lead @ s if tail is None else ((lead @ s.reshape(lead.shape[1], -1)) * tail).sum(-1)
            lo += cnt
        if K == 3:
            self.last = outs[2]
        return outs


def exact(case, seed):
    c = _full(case)
    if c["kind"] == "evaluate":
        e = _Exact(c, seed)
        x, T = e.x, c["T"]
        t = 0.5 * (_grid_xi(c["deg"]) + 1) * T
        tab = e.tables(_nodal(c, seed, x, t, 0)[0], 0).cpu()
        r = _rng(c, seed + 1)
        pts = np.concatenate([r.uniform(-1, 1, (c["npts"], c["dim"])), r.uniform(0, T, (c["npts"], 1))], 1)
        p = torch.from_numpy(pts)
        out = []
        P, Lt = tab.shape[1], _leg(c["deg"] + 1, 2 * p[:, 2] / T - 1)
        L0, L1 = _leg(P, p[:, 0]), _leg(P, p[:, 1])
        for k in range(2):
            w = (L0 @ tab[k].reshape(P, -1)).reshape(-1, P, c["deg"] + 1)
            out.append(((w * Lt[:, None, :]).sum(-1) * L1).sum(-1))
        return torch.stack(out, -1).numpy()
    # the rest within about 20 seconds: steps taken one after another, each some
    # hundred small operations (a thousand for the alpha-stable jump) over all paths
    evals = _evaluations(c) * c["iters"]
    P = c["n"] + 2
    cost = _longest(c) * (9e-3 if c["alpha"] < 2 else 1.5e-3 + 1.5e-4 * c["deg"]) + evals * (P * 3e-10 + 4.0 * P ** c["dim"] / 2e13)
    if c["kind"] not in ("step", "solve") or c["quad"] != "centre" or c["inst"] != 1 or cost > 20:
        return None
    e = _Exact(c, seed)
    h = lambda v: v.astype(np.float32) if c["prec"] == "fp32" else v  # noqa: E731
    shape = lambda U: U[None]  # noqa: E731
    if c["kind"] == "step":
        t = 0.5 * (_grid_xi(c["deg"]) + 1) * c["T"]
        U = _nodal(c, seed, e.x, t, 0)[0]
        S, ssq = e.estimate(U, 0, 0)
        eps = S - U[:, 1:].T if c["est"] == "picard" else S
        new = U.copy()
        new[:, 1:] += eps.T
        return {"U": shape(new), "eps": eps.reshape(1, -1), "sumsq": ssq.reshape(1, -1)}
    U0, out = _initial(c, seed, e.x), []
    for iv in range(len(e.wl.degree)):
        U = e.start(U0, iv)
        for k in range(c["iters"]):
            S, _ = e.estimate(U, iv, k)
            U = U.copy()
            U[:, 1:] = S.T if c["est"] == "picard" else U[:, 1:] + S.T
        out.append(shape(U))
        U0 = U[:, -1]
    return out
