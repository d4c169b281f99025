"""The single-read pass at the edges of the row widths its tiles are cut for: whole tiles, one column less, one more.
Bounds as in test_gpu_pass_shapes.py, of a sum of at most 1.5e4 products; a quadratic form's value is a difference of sums of
the size of its gradient."""
import numpy as np
import pytest
import torch

import oracle
import paper_2203_16340_amd as L
import test_gpu_pass_shapes as shapes
from gpu_helpers import DEV, rel_err, to_dev

pytestmark = pytest.mark.gpu

LSQ, L1, LOGI = L.OBJ_LSQ, L.OBJ_LSQ_L1SPLIT, L.OBJ_LOGISTIC_L2
TILES = [(LSQ, np.float64, c) for c in (3072, 12288, 14336)] + [(LSQ, np.float32, c) for c in (3072, 6144, 12288, 14336)]
TILES += [(LOGI, np.float64, c) for c in (1536, 3072, 12288)] + [(LOGI, np.float32, c) for c in (3072, 4096, 6144, 8192, 12288)]
TILES += [(L1, np.float64, 3072), (L1, np.float32, 6144)]


@pytest.mark.parametrize("kind,dtype,cols", TILES)
@pytest.mark.parametrize("rows,more", [(517, 0), (517, -1), (517, 1), (2051, -4), (67, 4)])
def test_around_a_tile(kind, dtype, cols, rows, more):
    shapes._check(kind, rows, cols + more, dtype, pad=0, shift=abs(more) % 2)


@pytest.mark.parametrize("dtype,cols", [t[1:] for t in TILES if t[0] == LOGI])
@pytest.mark.parametrize("more", [0, -1])
def test_rejected_first_steps(dtype, cols, more):
    shapes.test_columns_after_a_rejected_first_trial_step(dtype, 517, cols + more)


@pytest.mark.parametrize("dtype,n", [(np.float64, n) for n in (1026, 2048, 2050, 3072, 3074, 4094)] +
                         [(np.float32, n) for n in (1028, 2048, 2052, 2601, 3071, 3072, 3073, 3076, 4092, 4095)])
def test_quadratic_form(dtype, n):
    rng = np.random.default_rng(n)
    K = rng.standard_normal((n, n)).astype(dtype)
    K = np.ascontiguousarray((K + K.T) / dtype(2))
    b, x = rng.standard_normal(n), rng.standard_normal(n)
    f_ref, g_ref, row_ref = oracle.fg(oracle.Objective(oracle.QP, K, b), x, want_rowvec=True)
    s = L.Solver(L.OBJ_QP, to_dev(K), to_dev(b), to_dev(np.full(n, -np.inf)), to_dev(np.full(n, np.inf)), 3)
    assert s.apass_name == "fused"
    f, g, row = s.dbg_fg(to_dev(x), want_rowvec=True)
    assert abs(f - f_ref) <= 1e-12 * max(abs(f_ref), np.linalg.norm(x) * np.linalg.norm(g_ref))
    assert rel_err(g.cpu().numpy(), g_ref) <= 1e-12
    assert rel_err(row.cpu().numpy(), row_ref) <= 1e-12
    s.close()


# both sides of the size up to which the matrix is left in the memory-side cache, for every family of kernels that reads it once
@pytest.mark.parametrize("kind,dtype,cols", [(LSQ, np.float64, 301), (LSQ, np.float32, 1000), (LSQ, np.float64, 3001), (LSQ, np.float32, 3000),
                                             (LSQ, np.float64, 22529), (L1, np.float32, 6001), (LOGI, np.float32, 100), (LOGI, np.float64, 701),
                                             (LOGI, np.float32, 3001), (LOGI, np.float64, 2000), (L.OBJ_QP, np.float64, None), (L.OBJ_QP, np.float32, None)])
@pytest.mark.parametrize("above", [False, True])
def test_around_the_cache_size(kind, dtype, cols, above):
    size = np.dtype(dtype).itemsize
    if cols is None:                                         # rows = cols; above: past the kernels that read half of it
        cols = rows = (16000 if above else 2048) if size == 8 else (16100 if above else 4092)
    else:
        rows = (1 << 28) // (size * cols) + (1 if above else 0)
    gen = torch.Generator(device=DEV).manual_seed(cols)
    A = torch.randn(rows, cols, generator=gen, device=DEV, dtype=torch.float64 if size == 8 else torch.float32)
    n = 2 * cols if kind == L1 else cols
    x = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * 0.4
    b = torch.randn(rows, generator=gen, device=DEV, dtype=torch.float64)
    if kind == LOGI:
        b = torch.where(b >= 0, 1.0, -1.0).double()
    if kind == L.OBJ_QP:
        A = ((A + A.T) / 2).contiguous()
    l, u = torch.zeros(n, dtype=torch.float64, device=DEV), torch.full((n,), np.inf, dtype=torch.float64, device=DEV)
    kw = dict(lam=0.3 if kind == L1 else 0.0, mu=1e-3 if kind == LOGI else 0.0)
    one, two = (L.Solver(kind, A, b, l, u, 5, options=L.default_options(tol=0.0, refresh_every=0, a_pass=p), **kw)
                for p in (L.APASS_AUTO, L.APASS_TWO_PASS))
    assert (one.apass_name, two.apass_name) == ("fused", "two_pass")
    (f1, g1, r1), (f2, g2, r2) = (s.dbg_fg(x, want_rowvec=True) for s in (one, two))
    assert abs(f1 - f2) <= 1e-12 * max(abs(f2), float(x.norm() * g2.norm()))
    assert float((g1 - g2).norm()) <= 1e-12 * float(g2.norm()) and float((r1 - r2).norm()) <= 1e-12 * float(r2.norm())
    if kind != L.OBJ_QP:                                     # (indefinite here)
        for s in (one, two):
            s.set_x(x)
            for _ in range(3):
                s.step(False)
        assert float((one.x() - two.x()).norm()) <= 1e-10 * float(two.x().norm())
    one.close(), two.close()


# the instantiations that stream the matrix (the tests on small matrices reach the other ones): whole tiles, and rows one element
# short of them, which start on any element
STREAMED = [(LSQ, np.float64, c) for c in (2048, 3072, 5120, 10240, 12288, 14336, 20428, 22528, 24576)]
STREAMED += [(LSQ, np.float32, c) for c in (2048, 3072, 5120, 6144, 10240, 12288, 14336, 20428)]
STREAMED += [(LOGI, np.float64, c) for c in (1024, 1536, 2048, 3072, 5120, 10240, 12288, 20428)]
STREAMED += [(LOGI, np.float32, c) for c in (2048, 3072, 4096, 5120, 6144, 8192, 10240, 12288, 20428)]
STREAMED += [(k, t, c * 16 // np.dtype(t).itemsize) for k in (LSQ, LOGI) for t in (np.float64, np.float32)
             for c in (8, 16, 24, 32, 48, 64, 96, 128, 192, 256, 320, 384)]


@pytest.mark.parametrize("kind,dtype,cols", STREAMED)
@pytest.mark.parametrize("less", [0, 1])
def test_streamed(kind, dtype, cols, less):
    test_around_the_cache_size(kind, dtype, cols - less, True)
