"""Edges of the work split: several direction pairs per FFT workgroup, cells
that hold several slices before they are flushed, and copied cells in narrow
grids.

Bars.  Fused against stored projections: the two differ in FP32 rounding
order and in the rounding of the fixed point (half a unit of 2^-18 per tap and
source, unbiased), 1e-6 of s_abs as in the other comparisons of the two.
Gradients against the FP64 oracle: 1e-4, the bar of the other adjoint tests;
values 2e-5, with six taps."""
import numpy as np
import pytest

import oracle as O
from helpers import rel_l2, err_scale, gpu_plan, to_dev, oracle_inputs, DEFAULT_T

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


def _fused_against_stored(cfg, T, window_w=4):
    import paper_2410_01316_amd as F
    x, y, w = to_dev(cfg["x"], cfg["y"], cfg["w"])
    out = []
    for w_in, mat in ((w, False), (w, True), (w.abs(), True)):
        plan = F.Plan(cfg["xi"], kernel=cfg["kernel"], n_ft=cfg["n_ft"], scale=cfg["scale"],
                      R=cfg["R"], T=T, window_w=window_w, materialize=mat,
                      n_max=cfg["x"].shape[0], m_max=cfg["y"].shape[0])
        out.append(plan(x, w_in, y).cpu().numpy())
        plan.check()
    e = err_scale(out[0], out[1], out[2])
    print("fused - stored %.2e" % e)
    return e


@pytest.mark.parametrize("scales", [(1, 1, 1, 1, 1, 1, 1, 1, 1, 1), (1, 1, 64, 64, 64, 64, 1, 8, 8, 8),
                                    (1, 0, 0, 1, 1, 0, 1, 1, 1, 1)], ids=["equal", "steps", "zeros"])
def test_cells_held_over_slices(scales):
    """Ten slices per direction and workgroup, scales equal or changing from
    one to the next; weights of one sign and size on a few points, so single
    cells come near the fixed point's bound."""
    N, S = 9 * 4096 + 11, 4096
    cfg = _cfg("gauss", 4, N, 65, 1500, 256, 1, 2.0)
    w = np.repeat(np.asarray(scales, float), S)[:N] * np.random.default_rng(2).choice([1.0, 0.999], N)
    cfg["w"] = w
    cfg["x"][: 5 * S] = cfg["x"][:3].repeat(5 * S // 3 + 1, 0)[: 5 * S]
    assert _fused_against_stored(cfg, DEFAULT_T["gauss"]) < 1e-6


@pytest.mark.parametrize("d", [3, 40])
@pytest.mark.parametrize("T", [0.22, 0.27, 0.285, 0.3, 0.32, 0.4])
def test_copied_cells_of_narrow_grids(T, d):
    """Grids of 256 cells with about 120 to 210 of them stored."""
    cfg = _cfg("energy", d, 9001, 70, 21, 128, d, 1.0)
    cfg["w"] *= np.random.default_rng(3).choice([-1.0, 1.0], 9001)
    assert _fused_against_stored(cfg, T) < 1e-6


@pytest.mark.parametrize("kernel,n_ft,d,M,P,W", [
    ("gauss", 128, 20, 2051, 4100, 4), ("gauss", 128, 40, 1027, 8200, 6),
    ("gauss", 256, 33, 3000, 2050, 8), ("energy", 1024, 7, 1500, 4003, 4),
    ("energy", 1024, 40, 1025, 2100, 6), ("laplace", 256, 40, 5000, 1501, 0)])
def test_runs_that_cross_tiles(kernel, n_ft, d, M, P, W):
    """More units of work than workgroups: runs that end inside a tile and
    cross into the next, values and all gradients, fused against stored."""
    cfg = _cfg(kernel, d, 301, M, P, n_ft, d, 1.5 * np.sqrt(d))
    v = np.random.default_rng(M).random(M) + 0.1
    res = []
    for mat in (False, True):
        plan = gpu_plan(cfg, grad=True, materialize=mat, window_w=W)
        x, y, w, vd = to_dev(cfg["x"], cfg["y"], cfg["w"], v)
        s = plan(x, w, y)
        gx, gy, gw = plan.grad(vd, want_x=True)
        plan.check()
        res.append([t.cpu().numpy() for t in (s, gy, gw, gx)])
    errs = [rel_l2(a, b) for a, b in zip(*res)]
    print("s %.2e grad_y %.2e grad_w %.2e grad_x %.2e" % tuple(errs))
    assert errs[0] < 1e-6 and errs[2] < 1e-6
    assert errs[1] < 5e-5 and errs[3] < 5e-5
