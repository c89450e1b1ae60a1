"""Table frames whose columns go sample by sample: a format bent too strongly for the sums, y turning at a
grid line, a window of 100 pixels or less under a fine grid.  A column's deposits are rounded once per run of equal
deposit row, whatever the number of its samples.  So under equal photons (roundings of one sign add up) a frame
of 250,000 samples a column is within an ordinary frame's error (4e-7 of the peak: FP32 window, fp16 hi + lo
deposits) of the oracle's at 250 a column, whose own sampling error (midpoint rule, 1000 samples a pixel) is 1e-7
at the most."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics
from workloads.synth import elliptical_gaussian_tables

pytestmark = pytest.mark.gpu

BENT = dict(nx=66, ny=50, grid=15, cx=[30.0, 30.0, 6.0, 2.0], cy=[22.0, 3.0, 4.0, -1.0])
CASES = {
    "bent": dict(BENT, a_column=250, dense=1000), "bent_f64": dict(BENT, a_column=250, dense=300, dtype=np.float64),
    # the middle one of five grid lines: 49 / 2
    "turning_on_a_grid_line": dict(a_column=250, dense=1000, nx=100, ny=50, grid=5, cx=[50.0, 47.0, 0.3],
                                   cy=[24.5, 0.0, 3.0]),
    "fine_grid": dict(a_column=250, dense=1000, nx=66, ny=50, grid=31, cx=[33.0, 31.0, 0.5], cy=[22.0, 9.0, 1.0]),
    # rows that end at any sample of a group, and columns of less than one
    "few": dict(BENT, a_column=5.1, dense=1), "very_few": dict(BENT, a_column=0.7, dense=1),
    "few_f64": dict(BENT, a_column=5.1, dense=1, dtype=np.float64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_frames_against_the_oracle(name):
    from tests import gpu_util
    c = dict(CASES[name])
    g, dtype, n = c["grid"], c.get("dtype", np.float32), int(c["a_column"] * 4 * c["nx"])
    psf = Psf(kind="table", gx=g, gy=g, kw=32, kh=32, os=4,
              tables=elliptical_gaussian_tables(np.random.default_rng(g), g, g, 32, 32, 4))

    def scene(n):
        tr = [Trace(0, 0, 0, 600.0, 603.0, n, c["cx"], c["cy"], 0.5, 0)]
        return Scene("table_singles", c["nx"], c["ny"], tr, psf, [np.full(n, 1.3, dtype)], "f32")

    print(f"case {name}", flush=True)
    o = oracle.render(scene(n), Request(rv_mps=-700.0, flux_scale=1e6 / n))
    n *= c["dense"]
    err = metrics.max_rel_err(gpu_util.render(scene(n), Request(rv_mps=-700.0, flux_scale=1e6 / n)), o)
    print(f"  err {err:.2e} of the peak", flush=True)
    assert err < 5e-7
