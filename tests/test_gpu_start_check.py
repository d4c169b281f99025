"""A start point that is refused leaves no trace: the steps behind it give the same bits as a solver's that was never asked.  Up to 32 768
variables the check and what follows it are enqueued together, beyond the host looks in between."""
import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v, dtype=np.float64)).to(DEV)


def make(kind, rows, cols, bad_matrix=False):
    rng = np.random.default_rng(rows + 3 * cols)
    A, opt = rng.standard_normal((rows, cols)) / np.sqrt(rows), {}
    n = {"l1": 2 * cols, "gauss": rows * cols, "entropy": rows * cols}.get(kind, cols)
    l, u = np.zeros(n), np.full(n, np.inf)
    b, x0 = rng.standard_normal(rows), 0.01 * rng.random(n)
    if kind == "qp":
        A = A.T @ A + 0.1 * np.eye(cols)
        b = rng.standard_normal(cols)
    elif kind == "logistic":
        b, l, opt = np.where(b > 0, 1.0, -1.0), np.full(n, -1.0), dict(mu=1e-3)
    elif kind == "l1":
        opt = dict(lam=0.05)
    elif kind == "extra":
        opt = dict(extra=(dev(np.ones((3, n))), dev(np.ones(3)), dev(np.full(3, 0.1))))
    elif kind in ("gauss", "entropy"):
        A, l, x0 = A - A.min(), np.full(n, 1e-9), (0.5 + rng.random(n)) / n
        b = np.concatenate([np.full(rows, 1 / rows), np.full(cols, 1 / cols)])
        opt = dict(lam=0.1, row_weight=dev(np.full(rows + cols, 4.0)))
    if bad_matrix:
        A[-1, -1] = np.inf
    which = {"lsq": L.OBJ_LSQ, "extra": L.OBJ_LSQ, "l1": L.OBJ_LSQ_L1SPLIT, "qp": L.OBJ_QP, "logistic": L.OBJ_LOGISTIC_L2,
             "gauss": L.OBJ_OT_GAUSS, "entropy": L.OBJ_OT_ENTROPY}[kind]
    return L.Solver(which, dev(A), dev(b), dev(l), dev(u), 4, options=L.default_options(tol=0.0), **opt), x0


CASES = [("lsq", 60, 20), ("lsq", 900, 301), ("lsq", 700, 2500), ("lsq", 9, 32768), ("lsq", 9, 32769), ("extra", 500, 700), ("l1", 300, 1025),
         ("qp", 40, 1500), ("logistic", 3000, 90), ("logistic", 900, 1100), ("gauss", 40, 70), ("entropy", 40, 70)]


@pytest.mark.parametrize("kind,rows,cols", CASES)
def test_refused_without_a_trace(kind, rows, cols):
    (s, x0), (t, _) = make(kind, rows, cols), make(kind, rows, cols)
    for bad, place in ((-5.0, 0), (float("nan"), len(x0) - 1), (-5.0, len(x0) // 2)):
        wrong = x0.copy()
        wrong[place] = bad
        with pytest.raises(L.LbfgsbError) as e:
            s.set_x(dev(wrong))                              # (before there is an iterate, and after one)
        assert e.value.code == L.E_INFEASIBLE_X0 and f"x0[{place}]" in str(e.value)
        if place == 0:
            with pytest.raises(L.LbfgsbError):
                s.step()
            s.set_x(dev(x0))
            t.set_x(dev(x0))
        for _ in range(3):
            s.step(False)
            t.step(False)
    assert torch.equal(s.x(), t.x()) and torch.equal(s.g(), t.g()) and s.info().as_dict() == t.info().as_dict()
    assert t.info().iters == 9
    s.close()
    t.close()


@pytest.mark.parametrize("kind,rows,cols", [c for c in CASES if c[0] not in ("gauss", "entropy")])
def test_a_gradient_that_is_not_finite(kind, rows, cols):
    s, x0 = make(kind, rows, cols, bad_matrix=True)
    with pytest.raises(L.LbfgsbError) as e:
        s.set_x(dev(x0))
    assert e.value.code == L.E_NONFINITE
    with pytest.raises(L.LbfgsbError):
        s.step()
    s.close()
