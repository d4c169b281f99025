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
    for s in (solved, waited, ahead):
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
    for _ in range(5):
        many.append(once(cores))
        one.append(once(cores[:1]))
    for xa, xb in zip(many[0][1], one[0][1]):
        assert torch.equal(xa, xb)
    assert min(t for t, _ in one) < 1.35 * min(t for t, _ in many)
    for s in solvers:
        s.close()
