"""Convergence confirmed on a gradient evaluated anew: by one workgroup up to 32 768 variables, by the Gram kernel beyond.  What the
solver then says of its free set against the same quantities formed here from its x and g: the number of fixed variables and the
maximum are exact, the norm is a sum of n squares (each order of adding them is within n 2^-53 of the true one)."""
import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kind,rows,cols", [("lsq", 3001, 63), ("lsq", 900, 1025), ("lsq", 40, 4097), ("lsq", 24, 32768),
                                            ("lsq", 24, 32769), ("l1", 900, 700), ("l1", 1500, 1301), ("qp", 1301, 1301)])
@pytest.mark.parametrize("uniform", [True, False])
def test_confirmed(kind, rows, cols, uniform):
    rng = np.random.default_rng(rows + cols)
    A = rng.standard_normal((rows, cols)) / np.sqrt(rows)
    n = 2 * cols if kind == "l1" else cols
    l, u = np.zeros(n), np.full(n, np.inf)
    if not uniform:
        u[rng.random(n) < 0.3] = 1e-2
    b = A @ np.where(rng.random(cols) < 0.05, rng.random(cols), 0.0) + 0.01 * rng.standard_normal(rows)
    if kind == "qp":
        A, b = A.T @ A + 0.1 * np.eye(n), -b
    which = {"lsq": L.OBJ_LSQ, "l1": L.OBJ_LSQ_L1SPLIT, "qp": L.OBJ_QP}[kind]
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to(DEV)
    o = L.default_options(tol=2e-2 if kind == "l1" else 1e-3, max_iter=2000)
    s = L.Solver(which, dev(A), dev(b), dev(l), dev(u), 5, lam=0.5 if kind == "l1" else 0.0, options=o)
    s.set_x(dev(np.zeros(n)))
    i = s.solve()
    assert i.status == L.CONVERGED and i.iters >= 2
    x, g = s.x().cpu().numpy(), s.g().cpu().numpy()
    fixed = ((x <= l + o.eps) & (g >= 0)) | ((x >= u - o.eps) & (g <= 0))
    assert i.n_fixed == fixed.sum()
    assert i.pg2 == pytest.approx(np.linalg.norm(g[~fixed]), rel=n * 2.0 ** -53)
    assert i.pginf == np.abs(x - np.clip(x - g, l, u)).max()
    assert s.info().as_dict() == i.as_dict()
    s.close()
