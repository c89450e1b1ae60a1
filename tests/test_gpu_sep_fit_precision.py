"""Accuracy of separable FP32 frames under the FP64 precision, where tiles and samples are enough for the
column nodes (1200^2: 722 tiles, 13.2 samples a pixel and more).  The FP64 per-sample sums such a frame had
before the nodes were off by 0.9e-7 to 1.4e-7 of the peak and 3.7e-8 to 5.6e-8 of the norm, of which the frame's
own rounding to FP32 makes 2.5e-8: no sum may leave more than 1.1e-7 and 3.7e-8 here (FP32 partials of 16
nodes: 1.2e-7 to 1.7e-7 and 4.3e-8 to 5.3e-8)."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("smin,smax,half", [(0.9, 1.3, 6), (1.0, 1.6, 8)])
@pytest.mark.parametrize("seed", [1, 2])
def test_no_further_from_the_oracle_than_fp64_sums(smin, smax, half, seed):
    from tests import gpu_util
    rng = np.random.default_rng(seed)
    n, nx, ny = 1100 * 22, 1200, 1200
    sig = rng.uniform(smin, smax, (5, 5, 2)).astype(np.float32)
    psf = Psf(kind="separable", gx=5, gy=5, half_width=half, sigma_xy=sig)
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.85 * q, 550.0, 3.0], [45.3 + 70.0 * q, 12.0, -4.0], 0.5, q)
           for q in range(16)]
    k = np.arange(n)
    spec = [(1e4 * rng.uniform(0.5, 1.5) * (1.0 + 0.9 * np.sin(k / rng.uniform(7, 60)))).astype(np.float32)
            for _ in trs]
    sc = Scene("sep_fit_precision", nx, ny, trs, psf, spec, "f32")
    rq = Request(rv_mps=700.0, flux_scale=1.7)
    print(f"case {smin} {smax} {half} {seed}", flush=True)
    g, o = gpu_util.render(sc, rq).astype(np.float64), oracle.render(sc, rq)
    d = g - o
    print("max", np.max(np.abs(d)) / o.max(), "norm", np.linalg.norm(d) / np.linalg.norm(o), flush=True)
    assert np.max(np.abs(d)) < 1.1e-7 * o.max()
    assert np.linalg.norm(d) < 3.7e-8 * np.linalg.norm(o)
