"""Performance cases of the library: the calls a program makes, over the range
of sizes, kernels, precisions and options they are made with.

A case is a dict of plain values.  `kind` is the entry point:

  matvec   amg_matvec: one FP64 product with the finest level
  vcycle   amg_vcycle: one V-cycle, the preconditioner of a caller's own loop
  solve    amg_solve with a handle the program keeps (stationary V-cycle
           iteration, CG or GMRES)
  bdf4     amg_bdf4_step: one implicit time step
  batch    amg_solve_batch over uneven instances
  request  amg_setup, amg_solve, amg_destroy: a problem that is solved once

N is the number of intervals.  The library takes powers of two only, so the
odd sizes are the unknown counts (2N - 1), the horizons (delta N is not an
integer) and the mixes of a batch.  Kernels: the constant one, the weighted
one with 1.2 / 0.8 (not symmetric: general spectra) and the fractional one.

`exact` evaluates the same products, cycles and solutions in FP64 with plain
torch, from the definition of the collocation rule and of the Galerkin levels.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2202_11288_amd import binding as B

WL, WR = 1.2, 0.8  # the weighted kernel's sides
COARSEST = 5       # log2 of the coarsest level's intervals (the default)
OMEGA = 2.0 / 3.0  # damping (the default)


def listed():
    return [
        # a product of a small problem inside a caller's own iteration: launch latency
        dict(name="matvec_2e8_const_f64", kind="matvec", logN=8, kernel="const", delta=0.25),
        # the largest size the library takes, general spectra: memory traffic
        dict(name="matvec_2e22_weighted_f64", kind="matvec", logN=22, kernel="weighted", delta=0.1),
        # one preconditioner application at the benchmark's size, FP32
        dict(name="vcycle_2e20_const_mixed", kind="vcycle", logN=20, kernel="const", delta=0.25,
             mixed=True, deep=False, m1=1, m2=1),
        # the same in FP64 for a non-symmetric operator of ordinary size, two sweeps a side
        dict(name="vcycle_2e17_weighted_f64", kind="vcycle", logN=17, kernel="weighted",
             delta=0.05, mixed=False, deep=False, m1=2, m2=2),
        # a small problem: every level runs in the small-level kernels
        dict(name="solve_2e10_const_f64", kind="solve", logN=10, kernel="const", delta=0.25,
             mixed=False, deep=False, inner="vcycle", tol=1e-10),
        # an ordinary problem of the plain configurations, non-symmetric
        dict(name="solve_2e16_weighted_mixed", kind="solve", logN=16, kernel="weighted",
             delta=0.05, mixed=True, deep=False, inner="vcycle", tol=1e-10),
        # the benchmark's workload
        dict(name="solve_2e20_const_mixed_deep", kind="solve", logN=20, kernel="const",
             delta=0.25, mixed=True, deep=True, inner="vcycle", tol=1e-10),
        # the largest size, conjugate gradients
        dict(name="solve_2e22_const_mixed_cg", kind="solve", logN=22, kernel="const", delta=0.25,
             mixed=True, deep=False, inner="pcg", tol=1e-10),
        # a non-symmetric operator by GMRES, FP64
        dict(name="solve_2e18_weighted_f64_gmres", kind="solve", logN=18, kernel="weighted",
             delta=0.25, mixed=False, deep=False, inner="gmres", tol=1e-10),
        # a time step of the diffusion problem
        dict(name="bdf4_2e13_const_f64", kind="bdf4", logN=13, kernel="const", delta=0.25,
             mixed=False, tol=1e-8),
        # many independent problems of uneven size in one call
        dict(name="batch_48_uneven_mixed_cg", kind="batch", count=48, lo=10, hi=16, mixed=True,
             pick=1, tol=1e-10),
        # a served request whose problem has not been seen before: its set-up counts
        dict(name="request_2e14_weighted_mixed", kind="request", logN=14, kernel="weighted",
             delta=0.13, mixed=True, deep=False, inner="vcycle", tol=1e-8),
    ]


def draw(rng):
    kind = rng.choice(["matvec", "vcycle", "vcycle", "solve", "solve", "solve", "bdf4", "batch",
                       "request"])
    if kind == "batch":
        lo = rng.randint(8, 12)
        return dict(kind=kind, count=rng.randint(5, 48), lo=lo, hi=rng.randint(lo, 16),
                    mixed=rng.random() < 0.7, pick=rng.randrange(1 << 20), tol=1e-10)
    lo, hi = {"matvec": (6, 22), "vcycle": (7, 22), "solve": (7, 20), "bdf4": (7, 18),
              "request": (10, 18)}[kind]
    case = dict(kind=kind, logN=rng.randint(lo, hi),
                kernel="const" if kind == "bdf4" else rng.choice(["const", "weighted"]),
                delta=rng.uniform(0.02, 0.3))
    if kind == "matvec":
        return case
    case["mixed"] = rng.random() < 0.6
    if kind == "bdf4":
        return dict(case, tol=1e-8)
    case["deep"] = kind != "request" and rng.random() < 0.3
    if kind == "vcycle":
        return dict(case, m1=rng.choice([1, 1, 2]), m2=rng.choice([1, 1, 2]))
    inner = "vcycle"
    if kind == "solve":
        inner = rng.choice(["vcycle", "pcg" if case["kernel"] == "const" else "gmres"])
    return dict(case, inner=inner, tol=rng.choice([1e-8, 1e-10]))


# ---- inputs -----------------------------------------------------------------

def instances(case):
    """The problems of a batch: N = 2^K, delta and the kernel drawn per instance."""
    g = np.random.default_rng(case["pick"])
    out = []
    for _ in range(case["count"]):
        frac = bool(g.integers(0, 2))
        out.append(dict(logN=int(g.integers(case["lo"], case["hi"] + 1)),
                        delta=float(g.uniform(0.05, 0.3)),
                        kernel="fractional" if frac else "const",
                        alpha=float(g.uniform(0.2, 0.3))))
    return out


def points(N):
    """The collocation points in the library's order: nodes, then midpoints."""
    return np.concatenate([np.arange(1, N) / N, (np.arange(N) + 0.5) / N])


def smooth(N, g, modes=4):
    """A forcing term as a discretised problem has: a few sine modes."""
    x = points(N)
    return sum(g.standard_normal() / k * np.sin(k * math.pi * x) for k in range(1, modes + 1))


def inputs(case, seed):
    """The host arrays of a case: right-hand sides or vectors, by kind."""
    g = np.random.default_rng(seed)
    if case["kind"] == "batch":
        return [g.standard_normal((2 << d["logN"]) - 1) for d in instances(case)]
    N = 1 << case["logN"]
    if case["kind"] in ("matvec", "request") or case.get("inner") == "gmres":
        return [g.standard_normal(2 * N - 1)]
    if case["kind"] == "vcycle":  # a residual: all frequencies, the smooth ones larger
        return [g.standard_normal(2 * N - 1) + 10 * smooth(N, g)]
    if case["kind"] == "solve":
        return [smooth(N, g)]
    # bdf4: four past levels of a decaying smooth solution, and the forcing
    tau, u, f = 1.0 / N, smooth(N, g), smooth(N, g)
    return [math.exp(-j * tau) * u for j in range(4)] + [tau * f]


def kernel_of(d):
    if d["kernel"] == "weighted":
        return B.kernel(B.AMG_K_WEIGHTED, wl=WL, wr=WR)
    if d["kernel"] == "fractional":
        return B.kernel(B.AMG_K_FRACTIONAL, alpha=d["alpha"])
    return B.kernel(B.AMG_K_CONST)


def options(case):
    o = dict(precision=B.AMG_MIXED if case.get("mixed") else B.AMG_FP64,
             m1=case.get("m1", 1), m2=case.get("m2", 1),
             flags=B.AMG_FLAG_DEEP_FOLD if case.get("deep") else 0,
             inner={"vcycle": B.AMG_INNER_VCYCLE, "pcg": B.AMG_INNER_PCG,
                    "gmres": B.AMG_INNER_GMRES}[case.get("inner", "vcycle")])
    if case["kind"] == "bdf4":
        o.update(shift=25.0 / 12.0, scale=1.0 / (1 << case["logN"]))
    if case["kind"] == "batch":
        o.update(inner=B.AMG_INNER_PCG, max_iter=1000)
    return B.amg_default_opts(**o)


class State:
    """The handles and vectors a program keeps; the handles go with it."""

    def __init__(self, case):
        self.case = case
        self.handles = []

    def __del__(self):
        for h in self.handles:
            B.amg_destroy(h)


def prepare(case, seed):
    s = State(case)
    s.opts = options(case)
    if case["kind"] == "batch":
        for d in instances(case):
            s.handles.append(B.amg_setup(kernel_of(d), d["delta"], 1 << d["logN"], s.opts))
        s.tols = [case["tol"]] * case["count"]
    else:
        s.kernel, s.N = kernel_of(case), 1 << case["logN"]
        if case["kind"] != "request":
            s.handles.append(B.amg_setup(s.kernel, case["delta"], s.N, s.opts))
    dtype = torch.float32 if case["kind"] == "vcycle" and case["mixed"] else torch.float64
    s.ins = [torch.from_numpy(a).to("cuda", dtype) for a in inputs(case, seed)]
    s.outs = [torch.zeros_like(a) for a in (s.ins if case["kind"] == "batch" else s.ins[:1])]
    return s


OK = (B.AMG_OK, B.AMG_NOT_CONVERGED)


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "matvec":
        B.amg_matvec(s.handles[0], s.ins[0], s.outs[0])
    elif kind == "vcycle":
        B.amg_vcycle(s.handles[0], s.ins[0], s.outs[0])
    elif kind == "solve":
        s.outs[0].zero_()
        status, _, _ = B.amg_solve(s.handles[0], s.ins[0], s.outs[0], case["tol"], allow=OK)
        return {"x": s.outs[0], "status": status}
    elif kind == "bdf4":
        status, _, _ = B.amg_bdf4_step(s.handles[0], s.ins[:4], s.ins[4], s.outs[0], case["tol"],
                                       allow=OK)
        return {"x": s.outs[0], "status": status}
    elif kind == "batch":
        torch._foreach_zero_(s.outs)
        status, _, _ = B.amg_solve_batch(s.handles, s.ins, s.outs, s.tols, allow=OK)
        return {"x": s.outs, "status": status}
    else:
        h = B.amg_setup(s.kernel, case["delta"], s.N, s.opts)
        try:
            s.outs[0].zero_()
            status, _, _ = B.amg_solve(h, s.ins[0], s.outs[0], case["tol"], allow=OK)
        finally:
            B.amg_destroy(h)
        return {"x": s.outs[0], "status": status}
    return s.outs[0]


# ---- what a pass cannot do without -------------------------------------------

def sweep_work(n, elem, sym):
    """One product with a level: each vector, Cross vector and spectrum once,
    and the FFTs of the packed signal."""
    L = 2 * (n + 1)
    return (11 if sym else 16) * n * elem, 10 * L * math.log2(L) + 16 * L


def solve_work(d, elem, sweeps, iters):
    """`iters` V-cycles of element size elem, each with an FP64 residual."""
    sym = d["kernel"] != "weighted"
    by, fl = sweep_work((1 << d["logN"]) - 1, 8, sym) if iters else (0, 0)
    for k in range(d["logN"], COARSEST, -1):
        b1, f1 = sweep_work((1 << k) - 1, elem, sym)
        by, fl = by + sweeps * b1, fl + sweeps * f1
    return max(iters, 1) * by, max(iters, 1) * fl


def work(case):
    elem = 4 if case.get("mixed") else 8
    if case["kind"] == "matvec":
        by, fl = sweep_work((1 << case["logN"]) - 1, 8, case["kernel"] != "weighted")
    elif case["kind"] == "vcycle":
        by, fl = solve_work(case, elem, case["m1"] + case["m2"], 0)
    else:
        by = fl = 0
        iters = 6 if case["kind"] == "bdf4" else 8 if case.get("inner") == "vcycle" else 5
        for d in instances(case) if case["kind"] == "batch" else [case]:
            b1, f1 = solve_work(d, elem, 2, iters)
            by, fl = by + b1, fl + f1
    return {"bytes": by, "flops": fl}


# ---- the same in FP64 from the definitions ---------------------------------

def stencil(d):
    """Row stencil W at half-step offsets -S..S (W[s + S]) of the shifted
    collocation rule: on each cell of the horizon the quadratic through the
    values at its ends and its middle, integrated against the kernel."""
    N, delta = 1 << d["logN"], d["delta"]
    h, reach = 1.0 / N, delta * N
    r = int(math.floor(reach))
    cells = r + (1 if reach > r else 0)
    k = np.arange(cells, dtype=np.float64)
    theta = np.ones(cells)
    if reach > r:
        theta[-1] = reach - r
    if d["kernel"] == "fractional":
        alpha = d["alpha"]
        beta = -1.0 - 2.0 * alpha
        c = (1.0 - alpha) * delta ** (2.0 * alpha - 2.0) * h ** (beta + 1.0)
        t, wt = np.polynomial.legendre.leggauss(24)
        tau = 0.5 * theta[:, None] * (t + 1.0)
        g = c * 0.5 * theta[:, None] * wt * (k[:, None] + tau + (k == 0)[:, None]) ** beta
        J = [(g * tau ** j).sum(1) for j in range(3)]
        for j in range(3):  # the first cell in closed form (its j = 0 moment is not used)
            J[j][0] = c * theta[0] ** (beta + j + 1) / (beta + j + 1)
        wl = wr = 1.0
    else:
        c = 1.5 / delta ** 3 * h
        J = [c * theta ** (j + 1) / (j + 1) for j in range(3)]
        wl, wr = (WL, WR) if d["kernel"] == "weighted" else (1.0, 1.0)
    side = np.zeros(2 * cells + 1)
    side[0:-1:2] += J[0] - 3 * J[1] + 2 * J[2]
    side[1::2] += 4 * J[1] - 4 * J[2]
    side[2::2] += -J[1] + 2 * J[2]
    S = 2 * cells
    W = np.zeros(2 * S + 1)
    W[S + 1:] = -wr * side[1:]
    W[:S] = -wl * side[:0:-1]
    W[S] = -math.fsum(W)  # the basis sums to one
    return W, S


class Level:
    """A level [A p B; q o z; C x D]: Toeplitz generators (offsets
    -(n-1)..n-1), the row and column of the middle unknown, and its product."""

    def __init__(self, n, a, b, c, d, p, q, x, z, o):
        self.n, self.gen, self.cross, self.o = n, (a, b, c, d), (p, q, x, z), float(o)
        L = self.L = 2 * (n + 1)
        self.spec = []
        for g in self.gen:
            col = torch.zeros(L, dtype=torch.float64, device=g.device)
            col[:n] = g[:n].flip(0)             # offsets 0, -1, .., -(n-1): first column
            col[L - n + 1:] = g[n:].flip(0)     # offsets n-1, .., 1
            self.spec.append(torch.fft.rfft(col))
        self.diag = torch.cat([a[n - 1].expand(n), a.new_tensor([self.o]), d[n - 1].expand(n)])

    def mv(self, u):
        n, L = self.n, self.L
        v, w, wo = u[:n], u[n + 1:], u[n]
        fv, fw = torch.fft.rfft(v, L), torch.fft.rfft(w, L)
        a, b, c, d = self.spec
        p, q, x, z = self.cross
        yv = torch.fft.irfft(a * fv + b * fw, L)[:n] + p * wo
        yw = torch.fft.irfft(c * fv + d * fw, L)[:n] + x * wo
        return torch.cat([yv, (q @ v + z @ w + self.o * wo).reshape(1), yw])

    def coarse(self):
        """R A P with R = 1/4 [1 2 1], P = 2 R^T on the whole vector."""
        n, (a, b, c, d), (p, q, x, z) = self.n, self.gen, self.cross
        m = (n - 1) // 2
        at = n - 1  # index of offset 0
        e = torch.arange(-(m - 1), m, device=a.device)
        i = torch.arange(m, device=a.device)
        toe = lambda g: sum(k * g[2 * e + s + at] for s, k in
                            zip(range(-2, 3), (0.125, 0.5, 0.75, 0.5, 0.125)))
        st = list(zip(range(3), (0.25, 0.5, 0.25)))
        col = lambda g, f, t: sum(k * (0.5 * g[n - 1 - (2 * i + s) + at] + f[2 * i + s]
                                       + 0.5 * t[-(2 * i + s) + at]) for s, k in st)
        row = lambda g, f, t: sum(2 * k * (0.25 * g[2 * i + s - (n - 1) + at] + 0.5 * f[2 * i + s]
                                           + 0.25 * t[2 * i + s + at]) for s, k in st)
        o = (0.25 * (0.5 * a[at] + p[n - 1] + 0.5 * b[-(n - 1) + at])
             + 0.5 * (0.5 * q[n - 1] + self.o + 0.5 * z[0])
             + 0.25 * (0.5 * c[n - 1 + at] + x[0] + 0.5 * d[at]))
        return Level(m, toe(a), toe(b), toe(c), toe(d), col(a, p, b), row(a, q, c),
                     col(c, x, d), row(b, z, d), o)


def finest(d, shift, scale, dev):
    n = (1 << d["logN"]) - 1
    W, S = stencil(d)

    def at(s):
        return torch.from_numpy(scale * np.where(np.abs(s) <= S, W[np.clip(s + S, 0, 2 * S)], 0.0)
                                + shift * (s == 0)).to(dev)
    e, i = np.arange(-(n - 1), n), np.arange(n)
    # half-step positions: node i at 2i + 2, the middle unknown at 1, midpoint j at 2j + 3
    return Level(n, at(2 * e), at(2 * e + 1), at(2 * e - 1), at(2 * e), at(-2 * i - 1),
                 at(2 * i + 1), at(-2 * i - 2), at(2 * i + 2), at(np.array([0]))[0])


class Cycle:
    def __init__(self, d, shift=0.0, scale=1.0, m1=1, m2=1):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.m1, self.m2 = m1, m2
        self.levels = [finest(d, shift, scale, self.dev)]
        while self.levels[-1].n + 1 > 1 << COARSEST:
            self.levels.append(self.levels[-1].coarse())
        last = self.levels[-1]
        eye = torch.eye(2 * last.n + 1, dtype=torch.float64, device=self.dev)
        self.inv = torch.linalg.inv(torch.stack([last.mv(col) for col in eye], 1))

    def __call__(self, b, l=0):
        lv = self.levels[l]
        if l == len(self.levels) - 1:
            return self.inv @ b
        u = OMEGA * b / lv.diag
        for _ in range(self.m1 - 1):
            u = u + OMEGA * (b - lv.mv(u)) / lv.diag
        r = b - lv.mv(u)
        e = self(0.25 * (r[0:-2:2] + 2 * r[1:-1:2] + r[2::2]), l + 1)
        u[1::2] += e
        u[0:-2:2] += 0.5 * e
        u[2::2] += 0.5 * e
        for _ in range(self.m2):
            u = u + OMEGA * (b - lv.mv(u)) / lv.diag
        return u

    def solve(self, b, sym, most=60):
        """To FP64 accuracy: conjugate gradients (symmetric) or the plain iteration."""
        A, x, r = self.levels[0].mv, torch.zeros_like(b), b.clone()
        p = rz = None
        for _ in range(most):
            z = self(r)
            if not sym:
                x = x + z
                r = b - A(x)
            else:
                new = r @ z
                p = z if p is None else z + (new / rz) * p
                rz, q = new, A(p)
                alpha = rz / (p @ q)
                x, r = x + alpha * p, r - alpha * q
            if float(r.norm()) <= 1e-15 * float(b.norm()):
                break
        return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        ins = inputs(case, seed)
        out = []
        for d, b in zip(instances(case), ins):
            c = Cycle(d)
            out.append(c.solve(torch.from_numpy(b).to(c.dev), True, 200))
        return {"x": out, "status": None}
    if kind == "bdf4":
        c = Cycle(case, 25.0 / 12.0, 1.0 / (1 << case["logN"]))
        u1, u2, u3, u4, src = (torch.from_numpy(a).to(c.dev) for a in inputs(case, seed))
        b = 4 * u1 - 3 * u2 + (4.0 / 3.0) * u3 - 0.25 * u4 + src
        # from the last level, as the step does: the increment is small
        return {"x": u1 + c.solve(b - c.levels[0].mv(u1), True), "status": None}
    c = Cycle(case, m1=case.get("m1", 1), m2=case.get("m2", 1))
    b = torch.from_numpy(inputs(case, seed)[0]).to(c.dev)
    if kind == "matvec":
        return c.levels[0].mv(b)
    if kind == "vcycle":
        return c(b.float().double() if case["mixed"] else b)
    return {"x": c.solve(b, case["kernel"] != "weighted"), "status": None}
