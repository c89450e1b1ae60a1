"""Separable FP32 frames of isolated bright samples on darkness: no photons are negative, so no pixel is, also far
in the tails of a narrow Gaussian, where the column nodes' interpolant may pass below zero.  Negative samples keep
their sign (a frame is linear in its spectra)."""
import numpy as np
import pytest

from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu


def _scene(sigma, half, sign=1.0, dtype=np.float32):
    rng = np.random.default_rng(3)
    nx = ny = 1500
    n = 40 * 1400
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.85 * q, 700.0, 4.0], [60.0 + 60.0 * q, 20.0, -3.0], 1.0, q)
           for q in range(22)]
    spec = []
    for _ in trs:
        s = np.zeros(n, dtype)
        s[rng.integers(0, n, 300)] = sign * 1e6
        spec.append(s)
    psf = Psf(kind="separable", gx=2, gy=2, half_width=half, sigma_xy=np.full((2, 2, 2), sigma, np.float32))
    return Scene("signs", nx, ny, trs, psf, spec, "f32")


@pytest.mark.parametrize("prec", ["f64", "f16_hilo"])
@pytest.mark.parametrize("sigma,half", [(0.6, 8), (0.7, 6), (0.85, 8), (0.95, 8), (1.2, 8)])
def test_no_negative_pixels(sigma, half, prec):
    from tests import gpu_util
    print(f"case signs {sigma} {half} {prec}", flush=True)
    f = gpu_util.render(_scene(sigma, half), Request(rv_mps=10.0, precision=prec))
    assert f.max() > 0 and f.min() >= 0


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_negative_samples_keep_their_sign(dtype):
    from tests import gpu_util
    print(f"case negative {dtype.__name__}", flush=True)
    rq = Request(rv_mps=10.0)
    f, g = gpu_util.render(_scene(0.6, 8, 1.0, dtype), rq), gpu_util.render(_scene(0.6, 8, -1.0, dtype), rq)
    assert g.min() == -f.max() and np.max(np.abs(f + g)) < 1e-18 * f.max()


def test_batch_of_every_kind_of_frame():
    """Per sample, 10 nodes, 12, and 12 of a narrow Gaussian: each kernel has its own queue."""
    from tests import gpu_util
    scs = [_scene(s, h) for s, h in ((0.5, 6), (1.2, 8), (0.85, 6), (0.6, 8), (0.6, 8), (1.2, 8))]
    lds = [gpu_util.P.Loaded(gpu_util.ctx(), sc) for sc in scs]
    for prec in ("f64", "bf16_hilo"):
        rqs = [Request(rv_mps=10.0 * i, flux_scale=1.0 + i, precision=prec) for i in range(len(scs))]
        print(f"case signs batch {prec}", flush=True)
        outs = gpu_util.render_batch(scs, rqs, lds)
        for sc, ld, rq, o in zip(scs, lds, rqs, outs):
            assert o.min() >= 0 and np.array_equal(o, gpu_util.render(sc, rq, loaded=ld))
    for ld in lds:
        ld.free()
