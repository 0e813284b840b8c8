"""GPU tests of calls at the limits of what the library takes: values that are not finite, the largest launches,
memory that a call may need, and which launch shapes and paths a call leaves behind."""
import numpy as np
import pytest
import torch

from paper_1908_07392_amd import mhlp
from paper_1908_07392_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("px,py", [(np.inf, None), (-np.inf, None), (None, -np.inf), (np.inf, np.inf), (np.inf, np.nan)])
def test_volume_points_at_infinity(px, py):
    """A point at infinity keeps its cluster from being left out of any sum: the values that are not finite are those
    of the sum over all pairs, and the others agree with it."""
    rng = np.random.default_rng(1)
    n, alpha, h = 13000, 12.0, 0.01
    x, y = rng.uniform(-1.5, 1.5, n), rng.uniform(-1.5, 1.5, n)
    x[4321] = x[4321] if px is None else px
    y[4321] = y[4321] if py is None else py
    w, f = np.full(n, 1.0 / n), rng.standard_normal(n)
    out = torch.empty(n, dtype=torch.float64, device="cuda:0")
    u = mhlp.volume_eval(_t(x), _t(y), _t(w), _t(f), alpha, h)[0].cpu().numpy()
    v = mhlp.volume_eval_noalloc(_t(x), _t(y), _t(w), _t(f), alpha, h, out).cpu().numpy()
    assert np.array_equal(np.isnan(u), np.isnan(v)) and np.array_equal(np.isposinf(u), np.isposinf(v))
    ok = np.isfinite(v)
    assert (np.abs(u[ok] - v[ok]) <= 1e-12 * np.abs(v[ok]).max(initial=0.0)).all()
