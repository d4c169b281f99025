"""log, log1p and the logistic function as the kernels evaluate them on the device (lbfgsb_dbg_elementary), against 80-bit
arithmetic on the host."""
import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

LOG, LOG1P, SIGMOID = 0, 1, 2
N = 400_000


def evaluate(which, x):
    xd = to_dev(x)
    y = torch.empty_like(xd)
    torch.cuda.synchronize()
    assert L.lib().lbfgsb_dbg_elementary(which, xd.numel(), xd.data_ptr(), y.data_ptr()) == L.OK
    return y.cpu().numpy()


def ulps(got, ref):
    """Largest distance from ref (long double) in units of the last place of a double."""
    _, e = np.frexp(ref.astype(np.float64))
    return float((np.abs(got.astype(np.longdouble) - ref) / np.ldexp(np.longdouble(1), e - 53)).max())


def arguments(lo, hi, logarithmic, seed):
    t = np.random.default_rng(seed).random(N)
    if not logarithmic:
        return lo + t * (hi - lo)
    sign = np.sign(lo)
    return sign * np.exp(np.log(sign * lo) + t * (np.log(sign * hi) - np.log(sign * lo)))


@pytest.mark.parametrize("lo,hi", [(1e-16, 1e-6), (-1e-16, -1e-6), (1e-9, 1e-7), (-1e-9, -1e-7)])
def test_log1p_of_small_arguments(lo, hi):
    """1 + x keeps few bits of x: what its rounding took away, divided by 1 + x, is as large as the result's last bits or larger."""
    x = arguments(lo, hi, True, 1)
    assert ulps(evaluate(LOG1P, x), np.log1p(x.astype(np.longdouble))) <= 0.7


def test_refused():
    x = to_dev(np.ones(4))
    assert L.lib().lbfgsb_dbg_elementary(3, 4, x.data_ptr(), x.data_ptr()) == L.E_INVALID_ARG
    assert L.lib().lbfgsb_dbg_elementary(LOG, 0, x.data_ptr(), x.data_ptr()) == L.E_INVALID_ARG
    assert L.lib().lbfgsb_dbg_elementary(LOG, 4, None, x.data_ptr()) == L.E_INVALID_ARG
