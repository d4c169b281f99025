"""The work this library is timed on: whole calls of its public entry points, over the range they are used in.

A case names a problem family, its sizes, the storage type of the matrix, the number m of stored pairs and how the
solver is called:

  call = "solve"    lbfgsb_set_x + lbfgsb_solve to the case's tolerance; `iters` is about how many iterations that takes
  call = "steps"    lbfgsb_set_x + exactly `iters` lbfgsb_step calls without a host round trip
  call = "auglag"   one lbfgsb_auglag_solve; `iters` is about how many inner iterations it takes in all

Inputs are drawn on the device from the seed alone, with the recipes of workloads.py (same distributions, other draw
order).  `exact` repeats the method in plain torch in 64 bits: every objective, gradient and Armijo difference from
scratch, the two-loop recursion as the paper prints it.
"""
from __future__ import annotations

import math

import torch

import paper_2203_16340_amd as L

DEVICE = "cuda:0"


def listed():
    return [
        # the smallest call: a fit of a hundred coefficients, solved to 1e-8 (the benchmark's smallest configuration)
        dict(name="nnls_200x100", family="nnls", rows=200, cols=100, dtype="f64", m=5, call="solve", iters=51),
        # an everyday table of a few thousand samples with an odd number of columns
        dict(name="nnls_3001x301", family="nnls", rows=3001, cols=301, dtype="f64", m=10, call="solve", iters=11),
        # the benchmark's default workload, time to the relative tolerance 1e-6
        dict(name="nnls_20000x5000", family="nnls", rows=20000, cols=5000, dtype="f64", m=10, call="solve", iters=16),
        # L1-regularised least squares, more columns than rows, 40000 variables
        dict(name="lasso_10000x20000", family="lasso", rows=10000, cols=20000, dtype="f64", m=10, call="steps", iters=16),
        # box-constrained logistic regression, dense features
        dict(name="logistic_200000x2000_f32", family="logistic", rows=200000, cols=2000, dtype="f32", m=10, call="solve", iters=14),
        # logistic regression on a tall table: a million samples, a hundred features of different scales
        dict(name="logistic_1000000x100_f32", family="logistic", rows=1000000, cols=100, dtype="f32", m=10, call="steps", iters=16),
        # a large single-precision problem whose rows do not start on 16-byte boundaries (odd number of columns)
        dict(name="nnls_50001x3001_f32", family="nnls", rows=50001, cols=3001, dtype="f32", m=10, call="steps", iters=10),
        # the largest: 8 GB of matrix, two-sided box, 20 pairs
        dict(name="nnls_100000x20000_f32", family="nnls", rows=100000, cols=20000, dtype="f32", m=20, call="steps", iters=10),
        # dual SVM: a kernel matrix and one equality constraint; the first two outer iterations
        dict(name="svm_10000", family="svm", rows=10000, cols=10000, dtype="f64", m=10, call="auglag", iters=14),
        # joint probability distribution, Gaussian regulariser: a million variables, two thousand constraints
        dict(name="transport_gauss_1000x1000", family="transport_gauss", rows=1000, cols=1000, dtype="f64", m=10, call="auglag", iters=39),
        # the same with the entropy regulariser and random marginals: two million variables
        dict(name="transport_entropy_2000x1000", family="transport_entropy", rows=2000, cols=1000, dtype="f64", m=10, call="auglag", iters=46),
        # budget-constrained non-negative least squares (sum of x given), the whole augmented Lagrangian run
        dict(name="simplex_8000x2000", family="simplex", rows=8000, cols=2000, dtype="f64", m=10, call="auglag", iters=85),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["nnls", "nnls", "nnls", "lasso", "logistic", "logistic", "svm", "transport_gauss",
                         "transport_entropy", "simplex"])
    dtype = rng.choice(["f64", "f32"])
    m = rng.choice([5, 10, 10, 20])
    if family == "nnls":                  # overdetermined, up to about 2 GB
        cols = _log_int(rng, 60, 16000)
        rows = min(int(cols * math.exp(rng.uniform(math.log(2.5), math.log(40.0)))), 400_000_000 // cols)
        call, iters = ("solve", 14) if rows >= 3 * cols else ("steps", 10)
    elif family == "lasso":
        cols = _log_int(rng, 500, 20000)
        rows = int(cols * rng.uniform(0.4, 1.0))
        call, iters = "steps", 12
    elif family == "logistic":            # tall tables of a few dozen to a few thousand features
        cols = _log_int(rng, 24, 4000)
        rows = min(_log_int(rng, 20_000, 1_000_000), 400_000_000 // cols)
        call, iters = "steps", 12
    elif family == "svm":
        rows = cols = _log_int(rng, 1000, 10000)
        call, iters = "auglag", 14
    elif family == "simplex":
        cols = _log_int(rng, 200, 4000)
        rows = int(cols * rng.uniform(3.0, 6.0))
        call, iters = "auglag", 85
    else:
        rows, cols = _log_int(rng, 250, 2000), _log_int(rng, 250, 1000)
        call, iters = "auglag", 39 if family == "transport_gauss" else 46
        m = rng.choice([5, 10, 10])
    return dict(family=family, rows=rows, cols=cols, dtype=dtype, m=m, call=call, iters=iters)


# ---- inputs ------------------------------------------------------------------------------------------------------

def _chunks(rows, cols):
    step = max(1, (1 << 27) // cols)
    return [(r, min(rows, r + step)) for r in range(0, rows, step)]


def _times(A, v):
    """A v in 64 bits."""
    return torch.cat([A[a:b].double() @ v for a, b in _chunks(*A.shape)])


def _times_t(A, w):
    """A^T w in 64 bits."""
    out = torch.zeros(A.shape[1], dtype=torch.float64, device=A.device)
    for a, b in _chunks(*A.shape):
        out += A[a:b].double().T @ w[a:b]
    return out


def _normal_pdf(t, mean, sd):
    return torch.exp(-0.5 * ((t - mean) / sd) ** 2)


def _inputs(case, seed):
    """The problem's arrays, all on the device."""
    dev = torch.device(DEVICE)
    gen = torch.Generator(device=dev)
    gen.manual_seed(1_000_003 * int(seed) + 17)
    rows, cols, family = case["rows"], case["cols"], case["family"]
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32

    def normal(*shape, dtype=torch.float64):
        return torch.randn(shape, dtype=dtype, device=dev, generator=gen)

    def uniform(*shape, dtype=torch.float64):
        return torch.rand(shape, dtype=dtype, device=dev, generator=gen)

    def full(n, value):
        return torch.full((n,), value, dtype=torch.float64, device=dev)

    d = {}
    if family == "nnls":
        d["A"] = normal(rows, cols, dtype=dtype)
        small = rows * cols <= 20000
        keep = torch.randperm(cols, device=dev, generator=gen)[int(round((0.5 if small else 0.8) * cols)):]
        x = full(cols, 0.0)
        x[keep] = normal(keep.numel()).abs() if small else uniform(keep.numel())
        d["b"] = _times(d["A"], x) + 0.01 * normal(rows)
        d["l"], d["u"] = full(cols, 0.0), full(cols, 1.0 if dtype == torch.float32 else math.inf)
    elif family == "lasso":
        d["A"] = normal(rows, cols, dtype=dtype) / math.sqrt(rows)
        keep = torch.randperm(cols, device=dev, generator=gen)[: max(1, cols // 100)]
        x = full(cols, 0.0)
        x[keep] = normal(keep.numel())
        d["b"] = _times(d["A"], x) + 0.01 * normal(rows)
        d["lam"] = 0.1 * float(_times_t(d["A"], d["b"]).abs().max())
        d["l"], d["u"] = full(2 * cols, 0.0), full(2 * cols, math.inf)
    elif family == "logistic":
        d["A"] = normal(rows, cols, dtype=dtype)
        score = _times(d["A"], normal(cols)) + 0.5 * normal(rows)
        d["b"] = torch.where(score >= 0.0, 1.0, -1.0).double()
        if cols < 500:                    # tabular features come in different scales
            d["A"] *= torch.pow(10.0, 0.3 * (2.0 * uniform(cols) - 1.0)).to(dtype)
        d["mu"] = 1e-3
        d["l"], d["u"] = full(cols, -0.5), full(cols, 0.5)
    elif family == "svm":
        y = full(rows, 1.0)
        y[1::2] = -1.0
        way = normal(20)
        X = normal(rows, 20) / math.sqrt(20.0) + 0.5 * y[:, None] * (way / way.norm())[None, :]
        sq = (X * X).sum(1)
        K = torch.exp(-(sq[:, None] + sq[None, :] - 2.0 * (X @ X.T)).clamp_(min=0.0))
        d["A"] = (0.5 * (K + K.T)).to(dtype).contiguous()
        d["sign"], d["C"], d["d"] = y, y.reshape(1, rows).clone(), full(1, 0.0)
        d["b"], d["l"], d["u"] = full(rows, -1.0), full(rows, 0.0), full(rows, 1.0)
    elif family == "simplex":
        A = normal(rows, cols, dtype=dtype)
        keep = torch.randperm(cols, device=dev, generator=gen)[: cols // 5]
        x = full(cols, 0.0)
        x[keep] = uniform(keep.numel())
        b = _times(A, x) + 0.01 * normal(rows)
        d["A"] = torch.cat([A, torch.ones((1, cols), dtype=dtype, device=dev)])
        d["b"] = torch.cat([b, x.sum().reshape(1)])
        d["l"], d["u"] = full(cols, 0.0), full(cols, math.inf)
    else:
        n = rows * cols
        if family == "transport_gauss":   # smooth marginals, cost their outer product
            where = uniform(6)
            t, s = (torch.arange(rows, device=dev) + 0.5) / rows, (torch.arange(cols, device=dev) + 0.5) / cols
            u = _normal_pdf(t.double(), 0.4 + 0.2 * where[0], 0.10 + 0.05 * where[1])
            v = (_normal_pdf(s.double(), 0.25 + 0.1 * where[2], 0.05 + 0.02 * where[3])
                 + _normal_pdf(s.double(), 0.65 + 0.1 * where[4], 0.07 + 0.02 * where[5]))
            u, v = u / u.sum(), v / v.sum()
            M = torch.outer(u, _normal_pdf(s.double(), 0.5, 0.12) / cols)
            low = 0.0
        else:
            u, v = uniform(rows), uniform(cols)
            u, v = u / u.sum(), v / v.sum()
            M = uniform(rows, cols)
            low = 1e-30
        d["A"], d["d"] = M.to(dtype).contiguous(), torch.cat([u, v])
        d["lam"], d["l"], d["u"] = 0.5, full(n, low), full(n, math.inf)
    d["x0"] = d["l"].clone() if family.startswith("transport") else full(d["l"].numel(), 0.0)
    return d


def _options(case):
    """(options of the box solver, options of the augmented Lagrangian algorithm): the benchmark's settings, with the
    runs that take thousands of iterations cut to their first ones."""
    family, rows, cols = case["family"], case["rows"], case["cols"]
    if family == "svm":
        return dict(tol=1e-6 * math.sqrt(rows), max_iter=7), dict(ctol=1e-8, max_outer=2)
    if family == "transport_gauss":
        return dict(tol=1e-6, tol_relative=1, max_iter=39), dict(ctol=1e-6, max_outer=1)
    if family == "transport_entropy":
        return dict(tol=1e-4, tol_relative=1, max_iter=23, eps=1e-20), dict(ctol=1e-4, max_outer=2)
    if family == "simplex":
        return dict(tol=1e-4 * math.sqrt(rows)), dict(ctol=1e-8, max_outer=100)
    if case["call"] == "steps":
        return dict(tol=0.0, max_iter=100000), {}
    if rows * cols <= 20000:
        return dict(tol=1e-8), {}
    return dict(tol=1e-6, tol_relative=1), {}


def prepare(case, seed):
    d = _inputs(case, seed)
    box, outer = _options(case)
    options, family, m = L.default_options(**box), case["family"], case["m"]
    if family == "svm":
        s = L.AuglagRows(L.OBJ_QP, d["A"], d["b"], d["C"], d["d"], d["l"], d["u"], m, sign=d["sign"], options=options, **outer)
    elif family == "simplex":
        s = L.Auglag(d["A"], d["b"], 1, d["l"], d["u"], m, options=options, **outer)
    elif family.startswith("transport"):
        kind = L.OBJ_OT_GAUSS if family == "transport_gauss" else L.OBJ_OT_ENTROPY
        s = L.AuglagMarginals(kind, d["A"], d["d"], d["l"], d["u"], m, lam=d["lam"], options=options, **outer)
    else:
        kind = {"nnls": L.OBJ_LSQ, "lasso": L.OBJ_LSQ_L1SPLIT, "logistic": L.OBJ_LOGISTIC_L2}[family]
        s = L.Solver(kind, d["A"], d["b"], d["l"], d["u"], m, lam=d.get("lam", 0.0), mu=d.get("mu", 0.0), options=options)
    return dict(solver=s, x0=d["x0"], call=case["call"], iters=case["iters"])


def run(state):
    s = state["solver"]
    if state["call"] == "auglag":
        s.solve(state["x0"])
        return {"x": s.x(), "lambda": s.lam()}
    s.set_x(state["x0"])
    if state["call"] == "solve":
        info = s.solve()
        return {"x": s.x(), "f": info.f}
    for _ in range(state["iters"]):
        s.step(False)
    return {"x": s.x(), "g": s.g()}


def work(case):
    """One read of the matrix per evaluation at the start and per iteration.  Transport: no matrix product; the 2m
    stored vectors are read for the inner products and again for the direction, beside about eight vectors more."""
    rows, cols, iters = case["rows"], case["cols"], case["iters"]
    size = 8 if case["dtype"] == "f64" else 4
    if case["family"].startswith("transport"):
        n, v = rows * cols, 2 * case["m"] + 1
        return {"bytes": (iters * (2 * v + 8) + 4) * 8 * n, "flops": iters * n * (v * (v + 1) + 2 * v + 20)}
    products = 2 if case["family"] == "svm" else 4
    return {"bytes": (iters + 1) * rows * cols * size, "flops": (iters + 1) * products * rows * cols}


def tolerance(case):
    """All vectors, sums and products are 64-bit.  Measured against `exact` over the listed and 48 drawn cases: 1e-15 to
    4e-12 for plain solves and steps; the multipliers of a constrained run are small differences of sums, up to 6e-9."""
    return {"rel": 1e-7, "max": 4e-6} if case["call"] == "auglag" else {"rel": 2e-11, "max": 1e-9}


# ---- the same in plain torch, 64 bits, from scratch --------------------------------------------------------------

def _softplus(t):
    return t.clamp(min=0.0) + torch.log1p(torch.exp(-t.abs()))


class _Objective:
    """f + 0.5 rho ||C x - beta||^2 (marginals: C x = the row and column sums of the matrix x)."""

    def __init__(self, case, d):
        self.family, self.d, self.A = case["family"], d, d["A"]
        self.rows, self.cols = case["rows"], case["cols"]
        self.rho, self.beta = 0.0, None
        if self.family == "simplex":
            self.data, self.C, self.target = self.A[: self.rows], self.A[self.rows:].double(), d["b"][self.rows:]
            self.b = d["b"][: self.rows]
        else:
            self.data, self.C, self.target, self.b = self.A, d.get("C"), d.get("d"), d.get("b")

    def constraints(self, x):
        if self.family.startswith("transport"):
            P = x.reshape(self.rows, self.cols)
            return torch.cat([P.sum(1), P.sum(0)])
        return self.C @ x

    def spread(self, h):
        if self.family.startswith("transport"):
            return (h[: self.rows, None] + h[None, self.rows:]).reshape(-1)
        return self.C.T @ h

    def vector(self, x):
        if self.family == "lasso":
            return x[: self.cols] - x[self.cols:]
        return self.d["sign"] * x if self.family == "svm" else x

    def evaluate(self, x):
        """(gradient, what `difference` needs to know about x, objective)"""
        if self.family.startswith("transport"):
            M = self.A.double().reshape(-1)
            if self.family == "transport_gauss":
                g, f, at = M + self.d["lam"] * x, (M * x + 0.5 * self.d["lam"] * x * x).sum(), None
            else:
                logs = torch.log(x)
                g, f, at = M + self.d["lam"] * (logs + 1.0), (M * x + self.d["lam"] * x * logs).sum(), None
        else:
            z = _times(self.data, self.vector(x))
            if self.family == "logistic":
                y = self.b
                g = _times_t(self.data, -y * torch.sigmoid(-y * z)) / self.rows + self.d["mu"] * x
                f, at = _softplus(-y * z).mean() + 0.5 * self.d["mu"] * (x * x).sum(), z
            elif self.family == "svm":
                g = self.d["sign"] * z + self.b
                f, at = 0.5 * (self.vector(x) * z).sum() + (self.b * x).sum(), z
            else:
                at = z - self.b
                g, f = _times_t(self.data, at), 0.5 * (at * at).sum()
                if self.family == "lasso":
                    g, f = torch.cat([g, -g]) + self.d["lam"], f + self.d["lam"] * x.sum()
        h = None
        if self.rho:
            h = self.constraints(x) - self.beta
            g = g + self.rho * self.spread(h)
        return g, (at, h), float(f)

    def difference(self, x, xt, at):
        """f(xt) - f(x) without subtracting two objective values."""
        at, h = at
        dx = xt - x
        if self.family == "transport_gauss":
            df = (dx * (self.A.double().reshape(-1) + self.d["lam"] * (x + 0.5 * dx))).sum()
        elif self.family == "transport_entropy":
            near = dx.abs() <= 0.5 * x
            change = torch.where(near, dx * torch.log(xt) + x * torch.log1p(torch.where(near, dx / x, 0.0)),
                                 xt * torch.log(xt) - x * torch.log(x))
            df = (self.A.double().reshape(-1) * dx + self.d["lam"] * change).sum()
        else:
            dz = _times(self.data, self.vector(xt) - self.vector(x))
            if self.family == "logistic":
                q, dq = -self.b * at, -self.b * dz
                u = torch.sigmoid(q) * torch.expm1(dq)
                change = torch.where(u > -0.5, torch.log1p(u.clamp(min=-0.5)),
                                     torch.log(torch.sigmoid(-q) + torch.sigmoid(q) * torch.exp(dq)))
                df = change.mean() + 0.5 * self.d["mu"] * (dx * (xt + x)).sum()
            elif self.family == "svm":
                df = ((self.vector(xt) - self.vector(x)) * (at + 0.5 * dz)).sum() + (self.b * dx).sum()
            else:
                df = (dz * (at + 0.5 * dz)).sum()
                if self.family == "lasso":
                    df = df + self.d["lam"] * dx.sum()
        if self.rho:
            dh = self.constraints(dx)
            df = df + self.rho * (dh * (h + 0.5 * dh)).sum()
        return float(df)


def _two_loop(pairs, g, free, eps):
    q = torch.where(free, g, 0.0)
    kept = []
    for s, y, yy in reversed(pairs):
        ss, yf = torch.where(free, s, 0.0), torch.where(free, y, 0.0)
        rho = float(ss @ yf)
        if rho > eps * yy:
            alpha = float(ss @ q) / rho
            q = q - alpha * yf
            kept.append((ss, yf, rho, alpha, yy))
        else:
            kept.append(None)
    if kept and kept[0]:
        q = q * (kept[0][2] / kept[0][4])
    for k in reversed(kept):
        if k:
            q = q + (k[3] - float(k[1] @ q) / k[2]) * k[0]
    return -q


def _minimise(obj, l, u, x, m, tol, tol_relative=0, max_iter=1000, eps=1e-10):
    g, at, f = obj.evaluate(x)
    pairs, limit, done, converged = [], None, 0, False
    while True:
        free = ~(((x <= l + eps) & (g >= 0.0)) | ((x >= u - eps) & (g <= 0.0)))
        norm = float(torch.where(free, g, 0.0).norm())
        if limit is None:
            limit = tol * max(1.0, norm) if tol_relative else tol
        if norm <= limit or done >= max_iter:
            converged = norm <= limit
            break
        while True:
            d = _two_loop(pairs, g, free, eps)
            p = torch.minimum(torch.maximum(x + d, l), u) - x
            gp, pp, bound = float(p @ g), float(p @ p), 1.0
            if not (gp <= -eps * pp and pp >= eps):
                p = torch.where((d < 0.0) & (x <= l + eps) | (d > 0.0) & (x >= u - eps), 0.0, d)
                room = torch.where(p > 0.0, (u - x) / p, torch.where(p < 0.0, (l - x) / p, math.inf))
                gp, bound = float(p @ g), float(room.min())
            alpha, moved = min(1.0, bound), False
            for _ in range(61):
                xt = torch.minimum(torch.maximum(x + alpha * p, l), u)
                if obj.difference(x, xt, at) <= 1e-4 * alpha * gp:
                    moved = True
                    break
                alpha *= 0.5
            if moved or not pairs:
                break
            pairs = []
        if not moved:
            break
        gt, at, f = obj.evaluate(xt)
        pairs = (pairs + [(xt - x, gt - g, float((gt - g) @ (gt - g)))])[-m:]
        x, g, done = xt, gt, done + 1
    return x, g, f, converged


def exact(case, seed):
    d = _inputs(case, seed)
    obj, (box, outer) = _Objective(case, d), _options(case)
    l, u, x, m = d["l"], d["u"], d["x0"], case["m"]
    if case["call"] == "steps":
        x, g, _, _ = _minimise(obj, l, u, x, m, 0.0, max_iter=case["iters"])
        return {"x": x, "g": g}
    if case["call"] == "solve":
        x, _, f, _ = _minimise(obj, l, u, x, m, **box)
        return {"x": x, "f": f}
    lam, rho = torch.zeros_like(obj.target), 1.0
    before = float((obj.constraints(x) - obj.target).abs().max())
    for _ in range(outer["max_outer"]):
        obj.rho, obj.beta = rho, obj.target - lam / rho
        x, _, _, converged = _minimise(obj, l, u, x, m, **box)
        h = obj.constraints(x) - obj.target
        lam, now = lam + rho * h, float(h.abs().max())
        if now <= outer["ctol"] and converged:
            break
        if now > 0.5 * before:
            rho *= 2.0
        before = now
    return {"x": x, "lambda": lam}
