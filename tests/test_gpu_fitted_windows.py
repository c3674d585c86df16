"""Windows fitted to the kernel's spectrum (three taps for Gauss, five for
Laplace, on the general window's grid or a smaller one) against the FP64
oracle: the fused and the stored kernels, narrow and wide grids, the adjoint
and the batched form, with ragged point and direction counts.

Bars.  A fit is taken only where it moves the mean over the directions by
less than 5e-7 of the kernel's coefficients; with positive weights the sum
keeps more than a tenth of them, so the window adds at most 5e-6, and fixed
point and FP32 about as much: 2e-5.  The gradients keep the bar of the other
adjoint tests, 1e-4."""
import numpy as np
import pytest

import oracle as O
from helpers import rel_l2, gpu_plan, to_dev, oracle_inputs, DEFAULT_T

pytestmark = pytest.mark.gpu


def _cfg(kernel, d, N, M, P, n_ft, spread, seed):
    """Unit-variance points, positive weights, independent directions;
    `spread` is the kernel's width over the typical distance."""
    rng = np.random.default_rng(seed)
    x, y = rng.standard_normal((N, d)), rng.standard_normal((M, d))
    xi = rng.standard_normal((d, P))
    R = float(np.linalg.norm(x, axis=1).max() + np.linalg.norm(y, axis=1).max())
    return dict(x=x, y=y, w=rng.random(N) + 0.1, xi=xi / np.linalg.norm(xi, axis=0), kernel=kernel,
                scale=spread * np.sqrt(2.0 * d), n_ft=n_ft, R=R)


CASES = [
    # kernel, d, N, M, P, n_ft, spread, taps, cells
    ("gauss", 10, 67, 35, 3501, 512, 1.0, 3, 256),       # smaller grid than N_ft asks for
    ("gauss", 40, 97, 33, 2003, 512, 1.0, 3, 1024),   # the general window's grid, two k-blocks
    ("laplace", 5, 4097, 129, 130, 256, 1.0, 5, 512),
]


@pytest.mark.parametrize("materialize", [False, True], ids=["fused", "stored"])
@pytest.mark.parametrize("kernel,d,N,M,P,n_ft,spread,taps,cells", CASES)
def test_sum_matches_oracle(kernel, d, N, M, P, n_ft, spread, taps, cells, materialize):
    cfg = _cfg(kernel, d, N, M, P, n_ft, spread, seed=d)
    plan = gpu_plan(cfg, materialize=materialize)
    info = plan.info()
    assert (info["window_w"], info["n_grid"]) == (taps, cells)
    xd, yd, wd = to_dev(cfg["x"], cfg["y"], cfg["w"])
    s = plan(xd, wd, yd).cpu().numpy()
    plan.check()
    x, y, w, xi = oracle_inputs(cfg)
    tau = O.rescale_tau(kernel, cfg["R"], cfg["scale"], DEFAULT_T[kernel])
    e = rel_l2(s, O.kernel_sum_fourier(kernel, x, y, w, xi, cfg["scale"], n_ft, tau))
    print(f"{kernel} d={d} taps={taps} n={cells}: {e:.2e}")
    assert e < 2e-5


@pytest.mark.parametrize("materialize", [False, True], ids=["fused", "stored"])
def test_gradients_match_oracle(materialize):
    kernel, d, N, M, P, n_ft = "gauss", 33, 41, 50, 2003, 256
    cfg = _cfg(kernel, d, N, M, P, n_ft, 1.0, seed=7)
    plan = gpu_plan(cfg, grad=True, materialize=materialize)
    assert plan.info()["window_w"] == 3
    v = np.random.default_rng(8).random(M) + 0.1
    xd, yd, wd, vd = to_dev(cfg["x"], cfg["y"], cfg["w"], v)
    plan(xd, wd, yd)
    gx, gy, gw = (g.cpu().numpy() for g in plan.grad(vd, want_x=True))
    plan.check()
    x, y, w, xi = oracle_inputs(cfg)
    v = np.asarray(v, np.float32).astype(np.float64)
    tau = O.rescale_tau(kernel, cfg["R"], cfg["scale"], DEFAULT_T[kernel])
    a = (xi, cfg["scale"], n_ft, tau)
    errs = (rel_l2(gy, O.grad_y_fourier(kernel, x, y, w, *a) * v[:, None]),
            rel_l2(gw, O.grad_w_fourier(kernel, x, y, v, *a)),
            rel_l2(gx, O.grad_x_fourier(kernel, x, y, w, v, *a)))
    print("grad_y %.2e grad_w %.2e grad_x %.2e" % errs)
    assert max(errs) < 1e-4


@pytest.mark.parametrize("materialize", [False, True], ids=["fused", "stored"])
def test_batch_and_wide_window_agree(materialize):
    """More than one fixed-point slice, ragged tiles: three taps against the
    six-tap general window (within the bar above), and a batch whose problems
    all take three taps against the plans (equal up to the FP64 order of the
    sum over the directions)."""
    import paper_2410_01316_amd as F
    cfgs = [_cfg("gauss", d, N, M, 2003, 512, 1.0, seed=d) for d, N, M in
            ((10, 700, 1333), (40, 8200, 65), (3, 17, 1100))]
    ins = [to_dev(c["x"], c["w"], c["y"]) for c in cfgs]
    b = F.Batch([dict(xi=c["xi"], n_ft=c["n_ft"], scale=c["scale"], R=c["R"],
                      n_max=c["x"].shape[0], m_max=c["y"].shape[0]) for c in cfgs],
                kernel="gauss", materialize=materialize)
    outs = b(*zip(*ins))
    b.check()
    for c, (x, w, y), s in zip(cfgs, ins, outs):
        plan, wide = gpu_plan(c, materialize=materialize), gpu_plan(c, window_w=6)
        assert plan.info()["window_w"] == 3 and wide.info()["window_w"] == 6
        sp, sw = plan(x, w, y).cpu().numpy(), wide(x, w, y).cpu().numpy()
        print("d=%d: six taps %.2e batch %.2e" % (c["x"].shape[1], rel_l2(sp, sw),
                                                  rel_l2(s.cpu().numpy(), sp)))
        assert rel_l2(sp, sw) < 2e-5
        assert rel_l2(s.cpu().numpy(), sp) < 1e-6
