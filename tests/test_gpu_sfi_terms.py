"""Explicit fiber images of FP32 frames rendered as products of their terms,
at the edges of the path: sub-pixel counts 1 to 16, few and many terms,
smallest and largest windows, the narrowest accepted Gaussian, half discs,
traces over the detector's edges, one sample, FP64 spectra, and batches that
mix them with FP64 frames (rendered one by one)."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics

pytestmark = pytest.mark.gpu

# FP32 rounding of two operands, a scale, partial sums of 16 products and the
# output: at most about twelve half-ulps, 7e-7; the requirement on a frame is 1e-6
TOL = 1e-6


def _scene(n=120, nx=90, ny=50, rho=1.5, smin=0.8, smax=1.2, half=5, sub=10, shape="disc", grid=3, xh=30.0,
           cy=(24.3, 6.0), traces=2, dtype=np.float32, out="f32"):
    rng = np.random.default_rng(n + nx + sub)
    sig = rng.uniform(smin, smax, (grid, grid, 2)).astype(np.float32)
    psf = Psf(kind="sfi", gx=grid, gy=grid, half_width=half, sigma_xy=sig, fiber_radius=rho, fiber_shape=shape,
              subpix=sub)
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.3 * q, xh, 0.5], [cy[0] + 8.0 * q, *cy[1:]], 0.5, q)
           for q in range(traces)]
    spec = [(1e4 * rng.uniform(0.2, 1.5, n)).astype(dtype) for _ in range(traces)]
    return Scene("sfi_terms", nx, ny, trs, psf, spec, out)


CASES = {
    "one_sample": dict(n=1, traces=1), "paper": dict(), "centres_only": dict(sub=1), "two_sub": dict(sub=2),
    "sixteen_sub": dict(sub=16, n=60), "half_up": dict(shape="half_up"), "half_down": dict(shape="half_down"),
    "sixteen_terms": dict(rho=3.1, smin=0.78, smax=0.8, half=7, n=60),
    "few_terms": dict(rho=0.3), "window_3": dict(half=1, rho=0.4),
    "narrowest": dict(smin=0.581, smax=0.7, rho=1.2, sub=3),
    "off_edges": dict(xh=60.0, cy=(1.2, 3.0)), "ragged": dict(nx=129, ny=33, xh=63.0, cy=(20.0, 10.0), n=200),
    "chunk_edges": dict(n=64 + 13, traces=1), "f64_spectra": dict(dtype=np.float64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_frames_against_the_oracle(name):
    from tests import gpu_util
    sc = _scene(**CASES[name])
    rq = Request(rv_mps=-400.0, flux_scale=2.3)
    print(f"case {name}", flush=True)
    g, o = gpu_util.render(sc, rq), oracle.render(sc, rq)
    err = metrics.max_rel_err(g, o)
    print(f"  {err:.2e} of the peak", flush=True)
    assert err < TOL


def test_mixed_batch_equals_single_frames():
    from tests import gpu_util
    scs = [_scene(), _scene(out="f64"), _scene(smin=0.4, smax=0.6, rho=1.0), _scene(nx=129, ny=33, xh=60.0)]
    c = gpu_util.ctx()
    lds = [gpu_util.P.Loaded(c, sc) for sc in scs]
    rqs = [Request(rv_mps=5.0 * i, flux_scale=1.0 + i) for i in range(len(scs))]
    print("mixed batch", flush=True)
    outs = gpu_util.render_batch(scs, rqs, lds)
    for sc, rq, ld, o in zip(scs, rqs, lds, outs):
        assert np.array_equal(o, gpu_util.render(sc, rq, loaded=ld))
        assert metrics.max_rel_err(o, oracle.render(sc, rq)) < TOL
        ld.free()
