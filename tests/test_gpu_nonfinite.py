"""Non-finite inputs of the spread.  A source that is not finite and a NaN
weight add nothing (the point is reported by the bound check); projections
left behind a row's end by an earlier, longer call are never read as sources."""
import numpy as np
import pytest

from helpers import to_dev

pytestmark = pytest.mark.gpu

# kernel, d, n_ft, plan keywords: copies of cells, plain cells, wide grid, stored
PATHS = [("gauss", 3, 128, {}), ("gauss", 40, 1024, {}), ("energy", 5, 1024, {}),
         ("gauss", 3, 256, dict(materialize=True)), ("energy", 70, 1024, {})]
IDS = ["copies", "cells", "wide", "stored", "stored_gemm"]


def _plan(kernel, d, n_ft, kw, N, M):
    import paper_2410_01316_amd as F
    rng = np.random.default_rng(d)
    xi = rng.standard_normal((d, 37))
    xi /= np.linalg.norm(xi, axis=0)
    x, y, w = rng.standard_normal((N, d)), rng.standard_normal((M, d)), rng.random(N) + 0.1
    R = 1.01 * float(np.linalg.norm(x, axis=1).max() + np.linalg.norm(y, axis=1).max())
    make = lambda: F.Plan(xi, kernel=kernel, n_ft=n_ft, scale=1.5 * np.sqrt(d), R=R, n_max=N,
                          m_max=M, **kw)
    return make, x, y, w


@pytest.mark.parametrize("kernel,d,n_ft,kw", PATHS, ids=IDS)
def test_nonfinite_sources_and_weights_add_nothing(kernel, d, n_ft, kw):
    import paper_2410_01316_amd as F
    make, x, y, w = _plan(kernel, d, n_ft, kw, 4500, 200)
    plan = make()
    bad = np.array([0, 5, 6, 1003, 4098, 4499])
    w0 = w.copy()
    w0[bad] = 0.0
    xd, yd, wd, w0d = to_dev(x, y, w, w0)
    ref = plan(xd, w0d, yd).cpu().numpy()
    plan.check()
    wn = w.copy()
    wn[bad] = np.nan
    assert np.array_equal(plan(xd, to_dev(wn)[0], yd).cpu().numpy(), ref)
    plan.check()
    for v in (np.nan, -np.nan, np.inf, -np.inf):
        xn = x.copy()
        xn[bad] = v
        s = plan(to_dev(xn)[0], wd, yd).cpu().numpy()
        assert np.array_equal(s, ref), v
        with pytest.raises(F.FastSumError):
            plan.check()


@pytest.mark.parametrize("kernel,d,n_ft,kw", PATHS, ids=IDS)
def test_rows_left_by_a_longer_call(kernel, d, n_ft, kw):
    make, x, y, w = _plan(kernel, d, n_ft, kw, 4101, 203)
    xn, yn = x.copy(), y.copy()
    xn[1001:], yn[101:] = np.nan, np.nan
    plan = make()
    plan(*to_dev(xn, w, yn))
    s = plan(*to_dev(x[:1001], w[:1001], y[:101])).cpu().numpy()
    fresh = make()(*to_dev(x[:1001], w[:1001], y[:101])).cpu().numpy()
    assert np.all(np.isfinite(s)) and np.array_equal(s, fresh)
