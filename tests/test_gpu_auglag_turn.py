"""Algorithm 4 between two inner solves: multipliers, penalty parameter, stopping test and the change of targets are one kernel's
work (with the gradient's shift in it for few and short rows, behind it otherwise), and the host goes on without waiting for it.

Three inner solves against the oracle's, for constraint rows passed separately (both forms) and marginals; runs are the same bit
for bit whatever the host's pace; every way a run can end; an object used again starts afresh.

Inner solves end at 1e-9, curvatures are of order one and more, so minimisers agree far below 1e-6 and multipliers, which are
rho times differences of constraint values, below 1e-5 (as in the other tests of this algorithm)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2203_16340_amd as L
import workloads
from gpu_helpers import DEV, rel_err, to_dev

pytestmark = pytest.mark.gpu


def rows_problem(kind, n, n_eq, rng):
    C = rng.standard_normal((n_eq, n)) / np.sqrt(n)
    x = np.abs(rng.standard_normal(n))
    A = rng.standard_normal((2 * n, n)) / np.sqrt(n)
    if kind == "lsq":
        return A, A @ x + 0.1 * rng.standard_normal(2 * n), C, C @ (0.9 * x)
    return A.T @ A, -rng.random(n), C, 0.1 * C @ x


# one workgroup up to 64 rows and 16384 entries, then two kernels
@pytest.mark.parametrize("kind", ["lsq", "qp"])
@pytest.mark.parametrize("n,n_eq", [(40, 1), (300, 2), (257, 40), (300, 60), (9000, 2)])
def test_separate_rows(kind, n, n_eq):
    if n == 9000:
        if kind == "qp":
            pytest.skip("the matrix would be large")
        rng = np.random.default_rng(n)
        A = np.zeros((60, n))
        A[:, ::150] = rng.standard_normal((60, 60))
        b, C = rng.standard_normal(60), np.zeros((n_eq, n))
        C[:, ::150] = rng.standard_normal((n_eq, 60))       # (on the objective's own columns: the multipliers are not zero)
        l, u, d = np.full(n, -1.0), np.full(n, 1.0), rng.standard_normal(n_eq)
    else:
        A, b, C, d = rows_problem(kind, n, n_eq, np.random.default_rng(n + n_eq))
        l, u = np.zeros(n), np.full(n, 10.0)
    okind, gkind = (oracle.LSQ, L.OBJ_LSQ) if kind == "lsq" else (oracle.QP, L.OBJ_QP)
    x0 = np.clip(np.zeros(n), l, u)
    opts = dict(tol=1e-9, max_iter=5000)
    obj = oracle.Objective(okind, A, b).set_constraints(C, d)
    x_ref, lam_ref, _, iref = oracle.auglag_solve(obj, l, u, x0, 8, oracle.default_options(**opts), ctol=1e-30, max_outer=3)
    al = L.AuglagRows(gkind, to_dev(A), to_dev(b), to_dev(C), to_dev(d), to_dev(l), to_dev(u), 8,
                      options=L.default_options(**opts), ctol=1e-30, max_outer=3)
    for _ in range(2):
        info = al.solve(to_dev(x0))
        assert info.outer == iref.outer == 3 and info.rho == iref.rho and info.status == L.MAX_ITER
        if n != 9000:                                   # (there the minimiser is not unique)
            assert rel_err(al.x().cpu().numpy(), x_ref) <= 1e-6
        assert rel_err(al.lam().cpu().numpy(), lam_ref) <= 1e-5
        assert info.f == pytest.approx(iref.f, rel=1e-6, abs=1e-9)
    al.close()


# a row in several pieces of 1024 columns, the last one ragged; few columns
@pytest.mark.parametrize("kind,okind", [(L.OBJ_OT_GAUSS, oracle.OT_GAUSS), (L.OBJ_OT_ENTROPY, oracle.OT_ENTROPY)], ids=["gauss", "entropy"])
@pytest.mark.parametrize("rows,cols", [(3, 2500), (40, 37), (300, 2)])
def test_marginals(kind, okind, rows, cols):
    rng = np.random.default_rng(rows)
    M, n = rng.random((rows, cols)), rows * cols
    u, v = rng.random(rows) + 0.1, rng.random(cols) + 0.1
    u, v = u / u.sum(), v / v.sum()
    low = 0.0 if kind == L.OBJ_OT_GAUSS else 1e-30
    l, ub = np.full(n, low), np.full(n, np.inf)
    opts = dict(tol=1e-9, max_iter=3000, eps=1e-20)
    obj = oracle.Objective(okind, M, lam=0.5).set_marginals(u, v)
    x_ref, lam_ref, _, iref = oracle.auglag_solve(obj, l, ub, l.copy(), 8, oracle.default_options(**opts), ctol=1e-30, max_outer=3)
    al = L.AuglagMarginals(kind, to_dev(M), to_dev(np.concatenate([u, v])), to_dev(l), to_dev(ub), 8, lam=0.5,
                           options=L.default_options(**opts), ctol=1e-30, max_outer=3)
    info = al.solve(to_dev(l))
    assert info.outer == iref.outer == 3 and info.rho == iref.rho
    assert rel_err(al.x().cpu().numpy(), x_ref) <= 1e-6
    assert rel_err(al.lam().cpu().numpy(), lam_ref) <= 1e-5
    assert info.f == pytest.approx(iref.f, rel=1e-6)
    al.close()


def test_repeated_runs_are_the_same_bit_for_bit():
    cp = workloads.simplex_lsq(1500, 400, seed=3, budget=20.0, m=10)
    A_s, b_s, n_eq, l_s, u_s, x0_s = L.stack_constraints(cp.A, cp.b, cp.C, cp.d, cp.E, cp.e, cp.l, cp.u, cp.x0)
    al = L.Auglag(to_dev(A_s), to_dev(b_s), n_eq, to_dev(l_s), to_dev(u_s), cp.m, options=L.default_options(tol=1e-7), ctol=1e-9)
    x0, first = to_dev(x0_s), None
    busy = torch.randn(2048, 2048, device=DEV)
    for k in range(12):
        if k % 3 == 1:
            side = torch.cuda.Stream()                  # (another stream's work slows this one down)
            with torch.cuda.stream(side):
                for _ in range(20):
                    busy = busy @ busy * 1e-3
        info = al.solve(x0)
        got = info.as_dict(), al.x().clone(), al.lam().clone()
        assert info.status == L.CONVERGED and info.violation <= 1e-9
        if first is None:
            first = got
        assert got[0] == first[0] and torch.equal(got[1], first[1]) and torch.equal(got[2], first[2]), k
    torch.cuda.synchronize()
    al.close()


def test_a_line_search_that_fails_ends_the_run():
    n = 12
    A, b = 10.0 * np.eye(n), np.full(n, 100.0)
    C, d = np.ones((1, n)), np.array([3.0])
    for max_outer in (1, 5):
        al = L.AuglagRows(L.OBJ_LSQ, to_dev(A), to_dev(b), to_dev(C), to_dev(d), to_dev(np.full(n, -50.0)), to_dev(np.full(n, 50.0)), 4,
                          options=L.default_options(max_backtracks=0), max_outer=max_outer)
        info = al.solve(to_dev(np.zeros(n)))
        assert info.status == L.LINESEARCH_FAILED and info.outer == 1 and info.inner_iters == 0
        assert info.violation == 3.0 and info.rho == 1.0
        al.close()


def test_inner_solves_at_the_iteration_limit():
    A, b, C, d = rows_problem("lsq", 200, 2, np.random.default_rng(9))
    l, u = np.zeros(200), np.full(200, 10.0)
    obj = oracle.Objective(oracle.LSQ, A, b).set_constraints(C, d)
    for max_iter in (0, 1, 4):
        opts = dict(tol=1e-12, max_iter=max_iter)
        x_ref, lam_ref, _, iref = oracle.auglag_solve(obj, l, u, np.zeros(200), 5, oracle.default_options(**opts), ctol=1e-30, max_outer=6)
        al = L.AuglagRows(L.OBJ_LSQ, to_dev(A), to_dev(b), to_dev(C), to_dev(d), to_dev(l), to_dev(u), 5,
                          options=L.default_options(**opts), ctol=1e-30, max_outer=6)
        info = al.solve(to_dev(np.zeros(200)))
        assert info.outer == 6 and info.status == L.MAX_ITER and info.inner_iters == 6 * max_iter and info.rho == iref.rho
        assert rel_err(al.x().cpu().numpy(), x_ref) <= 1e-9 if max_iter else not al.x().any()
        assert rel_err(al.lam().cpu().numpy(), lam_ref) <= 1e-9
        al.close()


def test_no_constraint_rows():
    """Nothing to turn: one outer iteration, by the resident solver and by the others."""
    rng = np.random.default_rng(2)
    for rows, cols in ((60, 20), (900, 300)):
        A = rng.standard_normal((rows, cols))
        b = rng.standard_normal(rows)
        al = L.AuglagRows(L.OBJ_LSQ, to_dev(A), to_dev(b), torch.empty((0, cols), dtype=torch.float64, device=DEV),
                          torch.empty(0, dtype=torch.float64, device=DEV), to_dev(np.zeros(cols)), to_dev(np.full(cols, np.inf)), 5,
                          options=L.default_options(tol=1e-9))
        info = al.solve(to_dev(np.zeros(cols)))
        assert info.status == L.CONVERGED and info.outer == 1 and info.violation == 0.0
        x = al.x().cpu().numpy()
        assert np.abs(x - np.maximum(x - A.T @ (A @ x - b), 0.0)).max() <= 1e-8
        al.close()


@pytest.mark.parametrize("n,n_eq", [(3, 1), (40, 2), (9000, 2)])
@pytest.mark.parametrize("stacked", [True, False])
def test_a_subproblem_that_is_not_finite(n, n_eq, stacked):
    """Rows that cannot be met, from a penalty parameter that overflows f after some turns: with stacked rows the line search fails and
    the run ends with what it has, with separate rows it is refused as a start point would be."""
    rng = np.random.default_rng(n)
    A, b, C, d = rng.standard_normal((4, n)), np.ones(4), np.ones((n_eq, n)), np.full(n_eq, 2.0 * n)
    l, u = to_dev(np.zeros(n)), to_dev(np.ones(n))
    opts = dict(options=L.default_options(tol=1e-6, max_iter=20), rho0=1e300)
    if stacked:
        al = L.Auglag(to_dev(np.vstack([A, C])), to_dev(np.concatenate([b, d])), n_eq, l, u, 4, **opts)
        info = al.solve(u)
        assert info.status == L.LINESEARCH_FAILED and 10 < info.outer < 40 and info.violation == n and np.isinf(info.L)
        assert info.rho == 1e300 * 2.0 ** (info.outer - 1) and torch.equal(al.x(), u)
    else:
        al = L.AuglagRows(L.OBJ_LSQ, to_dev(A), to_dev(b), to_dev(C), to_dev(d), l, u, 4, **opts)
        with pytest.raises(L.LbfgsbError) as e:
            al.solve(u)
        assert e.value.code == L.E_NONFINITE
    al.close()
