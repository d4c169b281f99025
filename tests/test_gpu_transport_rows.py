"""The transport kinds' gradient and entropy update where their workgroups change: one, two and four rows each (512 and 1024
rows), 256 and 512 threads (384 columns), a last group of rows that is not full, one row, one column; few rows, whose columns
several workgroups share (up to 256 rows, the last workgroup's share empty or ragged); few columns, of which several rows fit
into a workgroup (up to 128: whole, ragged and 16 lanes, and the three row counts there); the whole-kernel sums
without a closing step.  Tolerances as in test_gpu_transport.py."""
import numpy as np
import pytest

import oracle
import paper_2203_16340_amd as L
from gpu_helpers import rel_err, to_dev
from test_gpu_transport import KIND_IDS, KINDS, _problem, _solver

pytestmark = pytest.mark.gpu

SHAPES = [(512, 384), (513, 385), (1023, 40), (1025, 386), (1030, 513), (1, 600), (700, 1), (2051, 70),
          (3, 5121), (16, 5000), (255, 1030), (256, 1024), (130, 128), (130, 129), (17000, 16), (9000, 17), (33000, 3), (4100, 65)]


@pytest.mark.parametrize("kinds", KINDS, ids=KIND_IDS)
@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("dtype", [np.float64, np.float32], ids=["f64", "f32"])
def test_value_and_gradient(kinds, rows, cols, dtype):
    kind, okind = kinds
    rng = np.random.default_rng(rows * 7 + cols)
    M, u, v = _problem(rng, rows, cols, dtype)
    n, lam, rho = rows * cols, 0.5, 2.5
    mult = rng.standard_normal(rows + cols)
    ref = oracle.Objective(okind, M, lam=lam).set_marginals(u, v, lam=mult, rho=rho)
    x = rng.random(n) / n + 1e-6
    f_ref, g_ref = oracle.fg(ref, x)
    s = _solver(kind, M, np.full(n, 1e-30), np.full(n, np.inf), 3, lam, np.concatenate([u, v]) - mult / rho, np.full(rows + cols, rho))
    for _ in range(3):                                    # (the sums start from scratch every time)
        f, g = s.dbg_fg(to_dev(x))
        assert abs(f - f_ref) <= 1e-12 * max(abs(f_ref), 1e-3)
        assert rel_err(g.cpu().numpy(), g_ref) <= 1e-12
    s.close()


@pytest.mark.parametrize("rows,cols", [(513, 385), (1025, 386), (1, 600), (700, 1), (2051, 70), (3, 5121), (255, 1030), (17000, 16),
                                       (4100, 65)])
@pytest.mark.parametrize("uniform", [True, False])
def test_entropy_iterations(rows, cols, uniform):
    rng = np.random.default_rng(rows + 3 * cols)
    M, u, v = _problem(rng, rows, cols)
    n, lam, rho = rows * cols, 0.5, 4.0
    mult = 0.01 * rng.standard_normal(rows + cols)
    l, ub = np.full(n, 1e-30), np.full(n, np.inf)
    if not uniform:
        ub[rng.random(n) < 0.1] = 2.0 / n
    x0 = np.where(rng.random(n) < 0.5, 1e-30, rng.random(n) / n)
    ref = oracle.Solver(oracle.Objective(oracle.OT_ENTROPY, M, lam=lam).set_marginals(u, v, lam=mult, rho=rho), l, ub, x0, 5,
                        oracle.default_options(tol=0.0))
    s = _solver(L.OBJ_OT_ENTROPY, M, l, ub, 5, lam, np.concatenate([u, v]) - mult / rho, np.full(rows + cols, rho), tol=0.0)
    s.set_x(to_dev(x0))
    for it in range(6):
        ref.step()
        info = s.step()
        assert info.branch == ref.info.branch and info.backtracks == ref.info.backtracks, it
        assert info.f == pytest.approx(ref.info.f, rel=1e-10), it
        assert rel_err(s.x().cpu().numpy(), ref.x) <= 1e-8 and rel_err(s.g().cpu().numpy(), ref.g) <= 1e-8, it
    ref.close()
    s.close()
