"""Table frames, whose columns are summed in blocks of samples: from less than
one sample a column to several hundred, columns whose row changes, traces flat
on a row edge, node cells that change inside a column in x and in y (also where
y turns at a grid line), formats bent too strongly for the sums, ragged ends
and FP64 spectra.  The bound is the requirement on a frame, 1e-6 of its peak
(the fp16 hi + lo deposits leave 2.4e-7)."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics
from workloads.synth import elliptical_gaussian_tables

pytestmark = pytest.mark.gpu


def _scene(n, nx=203, ny=97, kw=32, grid=3, cy=(48.3, 3.0, -1.2), cx=None, dtype=np.float32, traces=2):
    rng = np.random.default_rng(kw + grid)
    psf = Psf(kind="table", gx=grid, gy=grid, kw=kw, kh=kw, os=4,
              tables=elliptical_gaussian_tables(rng, grid, grid, kw, kw, 4))
    cx = cx or [nx / 2, 0.47 * nx, 0.3]
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [cx[0] + 0.85 * q, *cx[1:]], [cy[0] + 9.0 * q, *cy[1:]], 0.5, q)
           for q in range(traces)]
    spec = [(1e4 * rng.uniform(0.2, 1.5, n)).astype(dtype) for _ in trs]
    return Scene("table_sums", nx, ny, trs, psf, spec, "f32")


CASES = {
    "few": dict(n=41), "below_one_a_column": dict(n=600), "one_block": dict(n=203 * 4 * 16),
    "block_and_one": dict(n=203 * 4 * 17), "dense": dict(n=203 * 4 * 130),
    "f64_spectra": dict(n=203 * 4 * 11 + 3, dtype=np.float64), "f64_dense": dict(n=203 * 4 * 60, dtype=np.float64),
    "steep": dict(n=203 * 4 * 20, cy=(48.3, 44.0)), "steep_down": dict(n=203 * 4 * 20, cy=(48.3, -44.0)),
    "flat_on_a_row_edge": dict(n=203 * 4 * 12, cy=(47.5,)), "flat_near_it": dict(n=203 * 4 * 12, cy=(47.5 - 1e-7, 1e-6)),
    "turning_on_a_row_edge": dict(n=203 * 4 * 40, cy=(47.5, 0.0, 6.0)),
    "cells_in_a_column": dict(n=203 * 4 * 12, grid=31, cy=(40.3, 20.0)),
    # the middle one of five grid lines: 96 / 2
    "turning_on_a_grid_line": dict(n=203 * 4 * 40, grid=5, cy=(48.0, 0.0, 6.0)),
    "flat_on_a_grid_line": dict(n=203 * 4 * 12, grid=5, cy=(48.0,)),
    "bent": dict(n=66 * 4 * 30, nx=66, ny=50, grid=15, cx=[30.0, 30.0, 6.0, 2.0], cy=(22.0, 3.0, 4.0, -1.0)),
    "high_degree": dict(n=203 * 4 * 9, cx=[101.0, 90.0, 2.0, 1.0, 0.6, 0.4], cy=(48.3, 6.0, 3.0, -2.0, 1.0, 0.5)),
    "off_edges": dict(n=240 * 4 * 11, cx=[101.0, 120.0, 1.0], cy=(2.2, 1.4, 0.8)),
}


@pytest.mark.parametrize("kw", [32, 48])
@pytest.mark.parametrize("name", list(CASES))
def test_frames_against_the_oracle(name, kw):
    from tests import gpu_util
    sc = _scene(kw=kw, **CASES[name])
    rq = Request(rv_mps=-700.0, flux_scale=1.7)
    print(f"case {name} {kw}", flush=True)
    g, o = gpu_util.render(sc, rq), oracle.render(sc, rq)
    assert metrics.max_rel_err(g, o) < 1e-6
