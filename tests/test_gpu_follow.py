"""lbfgsb_solve enqueues steps ahead of what it knows and follows the kernels' reports in pinned host memory.  What it
returns must not depend on how far ahead the host happened to be: the same bits, counts and records in every run, and the
same as steps that are waited for one by one."""
import os
import threading
import time

import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L
import workloads
from gpu_helpers import DEV, make_solver, to_dev
from test_gpu_linesearch import LOGISTIC_CASES

pytestmark = pytest.mark.gpu


def _lsq(rows, cols, seed=1):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((rows, cols))
    b = A @ np.abs(rng.standard_normal(cols)) + 0.1 * rng.standard_normal(rows)
    return A, b, np.zeros(cols), np.full(cols, np.inf)


@pytest.mark.parametrize("rows,cols,a_pass", [(600, 200, L.APASS_TWO_PASS), (3000, 300, L.APASS_AUTO), (4000, 1500, L.APASS_AUTO)])
def test_a_solve_that_starts_at_the_solution_evaluates_nothing(rows, cols, a_pass):
    """The first step ends the run with a gradient that lbfgsb_set_x has just computed from x: there is nothing to confirm.
    The second step, enqueued behind it, reports the end as well and must not be taken for the one that found it."""
    A, b, l, u = _lsq(rows, cols)
    s = make_solver(L.OBJ_LSQ, A, b, l, u, 5, tol=1e-6, a_pass=a_pass)
    s.set_x(to_dev(l))
    assert s.solve().status == L.CONVERGED
    x = s.x().clone()
    for _ in range(20):
        s.set_x(x)
        info = s.solve()
        assert (info.status, info.iters, info.fevals) == (L.CONVERGED, 0, 1)
    s.close()


def _records(s):
    return [tuple(r.as_dict().values()) for r in s.history()]


@pytest.mark.parametrize("case", range(len(LOGISTIC_CASES)))
def test_rejected_first_steps_leave_the_same_bits_however_far_ahead_the_host_was(case):
    """Logistic searches that backtrack: a rejected first trial step parks the solver, the steps behind it are enqueued
    again, and for a while steps take the longer launch sequence, which carries f with other roundings.  lbfgsb_solve, steps
    waited for one by one and steps that are all enqueued before the first look must agree in every record, bit for bit."""
    prob = workloads.logistic(dtype=np.float64, **LOGISTIC_CASES[case])
    iters = 40
    solved, waited, ahead = (L.solver_for_problem(prob, DEV, tol=0.0, max_iter=iters) for _ in range(3))
    end = solved.solve()
    while waited.step().status == L.RUNNING:
        pass
    for _ in range(2 * iters):
        ahead.step(want_info=False)
    want = _records(waited)
    assert sum(1 for r in waited.history() if r.backtracks > 0) >= 3
    assert waited.info().as_dict() == end.as_dict() == ahead.info().as_dict()
    for s in (solved, ahead):
        assert _records(s) == want
        assert torch.equal(s.x(), waited.x()) and torch.equal(s.g(), waited.g())
    # (the static entry point looks at the status every few steps)
    x = to_dev(prob.x0)
    static = L.solve_static(prob.kind, to_dev(prob.A), to_dev(prob.b), to_dev(prob.l), to_dev(prob.u), prob.m, x, lam=prob.lam,
                            mu=prob.mu, options=L.default_options(tol=0.0, max_iter=iters))
    assert static.as_dict() == end.as_dict() and torch.equal(x, waited.x())
    for s in (solved, waited, ahead):
        s.close()


LIMITS = [0, 1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 13, 31, 32, 33, 39, 40, 41, 47, 48, 49]   # reports: 1 2 3 4 8 12 .. 32 40 48


@pytest.mark.parametrize("kind", [L.OBJ_LSQ, L.OBJ_LOGISTIC_L2])
@pytest.mark.parametrize("cols", [300, 1100])
def test_iteration_limits_around_the_reporting_steps(kind, cols):
    """The run ends at its limit whether or not that step reports, with the bits of steps waited for one by one."""
    if kind == L.OBJ_LSQ:
        A, b, l, u = _lsq(2000, cols)
        A *= np.geomspace(1.0, 30.0, cols)        # (more iterations than the largest limit)
    else:
        prob = workloads.logistic(rows=2000, cols=cols, seed=3, dtype=np.float64, mu=1e-4, bound=50.0)
        A, b, l, u = prob.A, prob.b, prob.l, prob.u
        A *= np.geomspace(0.1, 3.0, cols)
    x0 = to_dev(np.clip(np.zeros(cols), l, u))
    A, b, l, u = to_dev(A), to_dev(b), to_dev(l), to_dev(u)

    def solver(limit):
        s = L.Solver(kind, A, b, l, u, 10, mu=1e-4 if kind != L.OBJ_LSQ else 0.0, options=L.default_options(tol=0.0, max_iter=limit))
        s.set_x(x0)
        return s

    for limit in LIMITS:
        walk, s = solver(limit), solver(limit)
        while walk.step().status == L.RUNNING:
            pass
        for _ in range(2):                        # (the second finds a solver that has stopped)
            info = s.solve()
            assert (info.status, info.iters) == (L.MAX_ITER, limit)
            assert info.as_dict() == walk.info().as_dict() and _records(s) == _records(walk)
            assert torch.equal(s.x(), walk.x()) and torch.equal(s.g(), walk.g())
        s.close()
        walk.close()


def test_solving_again_after_convergence_changes_nothing():
    A, b, l, u = _lsq(2000, 700)
    s = make_solver(L.OBJ_LSQ, A, b, l, u, 10, tol=1e-9, tol_relative=1)
    s.set_x(to_dev(l))
    first = s.solve()
    x = s.x().clone()
    again = s.solve()
    assert first.status == again.status == L.CONVERGED and first.iters == again.iters and first.f == again.f
    assert torch.equal(s.x(), x)
    s.close()


def test_a_confirmation_that_does_not_confirm():
    """The gradient carried by recurrence passes the test, the one recomputed from x does not: the run goes on from the
    recomputed one until both pass.  (A start far away, so that the first steps leave rounding in the residual that is large
    against the tolerance; no periodic recomputation.)"""
    A, b, l, u = _lsq(1500, 400)
    l = np.full(400, -np.inf)
    x0 = np.full(400, 1e9)
    tol = 1e-3
    s = make_solver(L.OBJ_LSQ, A, b, l, u, 10, tol=tol, refresh_every=0)
    s.set_x(to_dev(x0))
    info = s.solve()
    x = s.x().cpu().numpy()
    trials = sum(r.backtracks + 1 for r in s.history())
    confirmations = info.fevals - 1 - trials
    print("confirmations", confirmations, info.as_dict())
    assert info.status == L.CONVERGED and confirmations >= 2
    assert np.linalg.norm(A.T @ (A @ x - b)) <= tol * 1.01
    s.close()


def test_threads_that_share_a_core_do_not_wait_for_each_other():
    """Four solvers on streams and threads of their own: the same bits on one core as on all, and nearly the same time.  A
    thread that follows its run gives its core to those that have steps to enqueue (3000 x 1200, ms per solve and thread:
    5.8 on eight cores, on one 9.6 without that, 5.9 with it)."""
    cores = sorted(os.sched_getaffinity(0))
    if len(cores) < 8:
        pytest.skip("needs eight cores to compare with")
    A, b, l, u = _lsq(3000, 1200)
    solvers = []
    for k in range(4):
        with torch.cuda.stream(torch.cuda.Stream()):
            solvers.append(make_solver(L.OBJ_LSQ, A, b + k, l, u, 10, tol=1e-12, tol_relative=1))
    x0 = to_dev(l)
    torch.cuda.synchronize()

    def run(s):
        for _ in range(15):
            s.set_x(x0)
            s.solve()

    def once(use):
        os.sched_setaffinity(0, use)
        try:
            threads = [threading.Thread(target=run, args=(s,)) for s in solvers]
            start = time.perf_counter()
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            return time.perf_counter() - start, [s.x().cpu() for s in solvers]
        finally:
            os.sched_setaffinity(0, cores)

    many, one = [], []
    for k in range(5):                            # (another core each time: one of them may be somebody else's)
        many.append(once(cores))
        one.append(once([cores[k * len(cores) // 5]]))
    for xa, xb in zip(many[0][1], one[0][1]):
        assert torch.equal(xa, xb)
    assert min(t for t, _ in one) < 1.45 * min(t for t, _ in many)
    for s in solvers:
        s.close()
