"""Edges of the work split: several direction pairs per FFT workgroup.

Bars.  Gradients against the FP64 oracle: 1e-4, the bar of the other adjoint tests;
values 2e-5, with six taps."""
import numpy as np
import pytest

import oracle as O
from helpers import rel_l2, gpu_plan, to_dev, oracle_inputs, DEFAULT_T

pytestmark = pytest.mark.gpu


def _cfg(kernel, d, N, M, P, n_ft, seed, scale):
    rng = np.random.default_rng(seed)
    xi = rng.standard_normal((d, P))
    x, y = rng.standard_normal((N, d)), rng.standard_normal((M, d))
    R = float(np.linalg.norm(x, axis=1).max() + np.linalg.norm(y, axis=1).max())
    return dict(x=x, y=y, w=rng.random(N) + 0.1, xi=xi / np.linalg.norm(xi, axis=0), kernel=kernel,
                scale=scale, n_ft=n_ft, R=R)


@pytest.mark.parametrize("materialize", [False, True], ids=["fused", "stored"])
@pytest.mark.parametrize("P,n_ft", [(1, 16), (2, 32), (3, 64), (7, 128), (9, 256), (15, 512),
                                    (17, 512), (3, 1024)])
def test_fft_pairs_and_gradients(P, n_ft, materialize):
    d, N, M = 5, 61, 43
    cfg = _cfg("gauss", d, N, M, P, n_ft, P, 6.0)
    plan = gpu_plan(cfg, grad=True, materialize=materialize, window_w=6)
    v = np.random.default_rng(P).random(M) + 0.1
    xd, yd, wd, vd = to_dev(cfg["x"], cfg["y"], cfg["w"], v)
    s = plan(xd, wd, yd).cpu().numpy()
    gx, gy, gw = (g.cpu().numpy() for g in plan.grad(vd, want_x=True))
    plan.check()
    x, y, w, xi = oracle_inputs(cfg)
    v = np.asarray(v, np.float32).astype(np.float64)
    a = (xi, cfg["scale"], n_ft, O.rescale_tau("gauss", cfg["R"], cfg["scale"], DEFAULT_T["gauss"]))
    e = rel_l2(s, O.kernel_sum_fourier("gauss", x, y, w, *a))
    errs = (rel_l2(gy, O.grad_y_fourier("gauss", x, y, w, *a) * v[:, None]),
            rel_l2(gw, O.grad_w_fourier("gauss", x, y, v, *a)),
            rel_l2(gx, O.grad_x_fourier("gauss", x, y, w, v, *a)))
    print("s %.2e grad_y %.2e grad_w %.2e grad_x %.2e" % ((e,) + errs))
    assert e < 2e-5 and max(errs) < 1e-4
