"""CCF at the edges of its launches, against the oracle: smoothing windows on
both sides of the single-launch limit and wider than the template's end
regions, templates shorter than a workgroup's samples, more velocities than
threads and the fewest, a velocity grid whose reads do not fit LDS, slices
sharing templates, FP64 templates, and unusable columns."""
import numpy as np
import pytest

import oracle
from workloads import Request
from workloads.synth import _espresso

pytestmark = pytest.mark.gpu


def _scene(nx=300, n=30000, dtype=np.float32, n_sli=2):
    return _espresso(41, nx=nx, ny=260, orders=[80, 81], n_samp=n, gx=3, kwid=0, psf_kind="separable", name="ccf",
                     xh=0.46 * nx, y0=70.0, pitch=110.0, n_lines=300, a_scale=0.02, b_total=4.0, n_fib=1,
                     n_sli=n_sli, fiber_kind=("star",), spec_dtype=dtype)


CASES = {
    # half-windows 512 and 513 of n / span = 108.7 samples a pixel
    "widest_single_launch": dict(smooth=512.2 / 108.7), "three_launches": dict(smooth=513.4 / 108.7),
    "narrow": dict(smooth=0.02), "three_velocities": dict(nv=3, v0=-300.0, dv=300.0),
    "many_velocities": dict(nv=601, v0=-15000.0, dv=50.0),
    "wide_grid": dict(nv=81, v0=-1e6, dv=2.5e4), "short_template": dict(n=900, smooth=1.0),
    "f64_templates": dict(dtype=np.float64), "unsliced_odd": dict(n_sli=1, n=29999, nx=301),
    "flat_with_holes": dict(holes=True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_ccf_equals_the_oracle(name):
    from paper_2008_05858_amd import Loaded
    from tests import gpu_util
    from tests.test_gpu_loop import gpu_ccf
    kw = dict(CASES[name])
    sp, nv, v0, dv = kw.pop("smooth", 1.5), kw.pop("nv", 101), kw.pop("v0", -5000.0), kw.pop("dv", 100.0)
    holes = kw.pop("holes", False)
    sc = _scene(**kw)
    print(f"case {name}", flush=True)
    F = oracle.render(sc, Request(rv_mps=700.0))
    Ex, L = oracle.extract(sc, F, 4.5)
    flat = None
    if holes:
        flat = 1.0 + np.random.default_rng(3).random(Ex.shape)
        flat[:, 100:130] = 0.0
        flat[1, :] = -1.0
    Co, rvo = oracle.ccf(sc, Ex, L, v0, dv, nv, flat=flat, smooth_px=sp)
    ld = Loaded(gpu_util.ctx(), sc)
    Cg, rvg = gpu_ccf(ld, sc, Ex, L, v0, dv, nv, flat=flat, smooth_px=sp)
    ld.free()
    assert np.max(np.abs(Cg - Co)) <= 1e-9 * np.abs(Co).max()
    assert abs(rvg - rvo) <= 1e-6 * abs(dv)
