"""lbfgsb_solve enqueues steps ahead of what it knows and follows the kernels' reports in pinned host memory.  What it
returns must not depend on how far ahead the host happened to be: the same bits, counts and records in every run, and the
same as steps that are waited for one by one."""
import numpy as np
import pytest

import paper_2203_16340_amd as L
from gpu_helpers import make_solver, to_dev

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
