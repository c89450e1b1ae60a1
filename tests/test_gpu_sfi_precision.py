"""Accuracy of explicit fiber images of FP32 frames: no further from their definition in 64 bits (chords by a
40-point rule, plain numpy) than the image-by-image FP64 sums were on the same four scenes."""
import numpy as np
import pytest
from scipy.special import ndtr

from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu

C = 299792458.0
# sub-pixels: largest error of the peak, error of the norm of those sums, measured on these scenes
BEFORE = {5: (1.142e-7, 4.688e-8), 10: (1.126e-7, 4.570e-8)}


def _exact(sc, rq):
    """Every sample's window: the sub-pixel means of the fiber's chords through its Gaussian, over their sum."""
    p, S, H = sc.psf, sc.psf.subpix, sc.psf.half_width
    R, n_win = p.fiber_radius, 2 * sc.psf.half_width + 1
    x40, w40 = np.polynomial.legendre.leggauss(40)
    th = 0.5 * np.pi * x40                       # chord at a = R sin(th), half length R cos(th)
    a, h, w = R * np.sin(th), R * np.cos(th), w40 * np.cos(th)
    lo = np.zeros(40) if p.fiber_shape == "half_up" else -h
    hi = np.zeros(40) if p.fiber_shape == "half_down" else h
    sub = (np.arange(S) + 0.5) / S - 0.5
    frame = np.zeros((sc.ny + 2 * n_win, sc.nx + 2 * n_win))
    for tr in sc.traces:
        lam = (tr.lmin + (np.arange(tr.n) + 0.5) * (tr.lmax - tr.lmin) / tr.n) * (1.0 + rq.rv_mps / C)
        t = (2.0 * lam - tr.lmin - tr.lmax) / (tr.lmax - tr.lmin)
        x, y = np.polynomial.polynomial.polyval(t, tr.cx), np.polynomial.polynomial.polyval(t, tr.cy)
        fx = np.clip(x * (p.gx - 1) / (sc.nx - 1), 0, p.gx - 1)
        fy = np.clip(y * (p.gy - 1) / (sc.ny - 1), 0, p.gy - 1)
        ix, iy = np.minimum(fx.astype(int), p.gx - 2), np.minimum(fy.astype(int), p.gy - 2)
        fx, fy = (fx - ix)[:, None], (fy - iy)[:, None]
        g = p.sigma_xy.astype(np.float64)
        sg = ((1 - fx) * g[iy, ix] + fx * g[iy, ix + 1]) * (1 - fy) + ((1 - fx) * g[iy + 1, ix] + fx * g[iy + 1, ix + 1]) * fy
        ax, ay = np.floor(x + 0.5).astype(int), np.floor(y + 0.5).astype(int)
        phi = sc.spectra[tr.slot].astype(np.float64) * tr.thr * rq.flux_scale
        d = np.arange(-H, H + 1)[:, None] + sub  # window pixel, sub-pixel
        for k in range(tr.n):
            u, v = (d - (x[k] - ax[k])) / sg[k, 0], d - (y[k] - ay[k])
            X = np.exp(-0.5 * (u[None] - a[:, None, None] / sg[k, 0]) ** 2).mean(2)
            Y = (ndtr((v[None] - lo[:, None, None]) / sg[k, 1]) - ndtr((v[None] - hi[:, None, None]) / sg[k, 1])).mean(2)
            W = (Y * w[:, None]).T @ X
            j, i = ay[k] - H + n_win, ax[k] - H + n_win
            frame[j:j + n_win, i:i + n_win] += phi[k] / W.sum() * W
    return frame[n_win:-n_win, n_win:-n_win]


@pytest.mark.parametrize("sub", [5, 10])
def test_no_further_off_than_image_by_image(sub):
    from tests import gpu_util
    worst, norm = 0.0, 0.0
    for seed, shape in enumerate(("disc", "half_up", "half_down", "disc")):
        rng = np.random.default_rng(seed)
        nx, ny, n = 300, 200, 700
        psf = Psf(kind="sfi", gx=5, gy=5, half_width=5, sigma_xy=rng.uniform(0.8, 1.2, (5, 5, 2)).astype(np.float32),
                  fiber_radius=1.5, fiber_shape=shape, subpix=sub)
        trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.3 * q, 140.0, 0.5], [25.3 + 20.0 * q, 6.0], 0.5, q)
               for q in range(8)]
        spec = [(1e4 * rng.uniform(0.5, 1.5, n)).astype(np.float32) for _ in trs]
        sc = Scene("sfi_precision", nx, ny, trs, psf, spec, "f32")
        rq = Request(rv_mps=-400.0, flux_scale=2.3)
        print(f"case {sub} {shape}", flush=True)
        g, o = gpu_util.render(sc, rq).astype(np.float64), _exact(sc, rq)
        worst = max(worst, np.max(np.abs(g - o)) / o.max())
        norm = max(norm, np.linalg.norm(g - o) / np.linalg.norm(o))
    print("worst", worst, "norm", norm, flush=True)
    assert worst <= BEFORE[sub][0] and norm <= BEFORE[sub][1]
