"""Separable FP32 frames rendered through column nodes, at the sizes where
that can go wrong: samples per column around the node count, both node
counts, a row anchor on the trace, sigma-grid lines in a column, ragged
widths, FP64 spectra, a trace of one or two samples, and batches that mix frames of
this path with frames of the per-sample kernels."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics

pytestmark = pytest.mark.gpu

# the requirement on a frame (1e-6 of the peak) for the FP64 and fp16 hi/lo
# variants, twice what the per-sample FP32 and bf16 hi/lo ones were measured at
BOUNDS = {"f64": 1e-6, "f32": 4e-6, "f16_hilo": 1e-6, "bf16_hilo": 3e-6}


def _scene(n, nx=203, ny=97, smin=1.0, smax=1.5, half=8, grid=3, cy=(48.3, 3.0, -1.2), xh=95.0,
           dtype=np.float32, seed=5, traces=2, bow=0.3, short=0):
    rng = np.random.default_rng(seed)
    sig = rng.uniform(smin, smax, (grid, grid, 2)).astype(np.float32)
    psf = Psf(kind="separable", gx=grid, gy=grid, half_width=half, sigma_xy=sig)
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.85 * q, xh, bow], [cy[0] + 9.0 * q, *cy[1:]], 0.5, q)
           for q in range(traces)]
    if short:
        trs[1].n = short
    spec = [(1e4 * rng.uniform(0.2, 1.5, t.n)).astype(dtype) for t in trs]
    return Scene("sep_fit", nx, ny, trs, psf, spec, "f32")


# (a frame of few tiles takes this path from 34 samples a pixel, one of 768
# and more from 14: the "wide" ones)
WIDE = dict(nx=3100, ny=520, xh=1500.0)
CASES = {
    "beside_a_one_sample_trace": dict(n=190 * 80, short=1), "beside_a_two_sample_trace": dict(n=190 * 80, short=2),
    "at_the_node_count": dict(n=3000 * 14, cy=(48.3, 30.0), bow=430.0, **WIDE),
    "above_the_node_count": dict(n=3000 * 17 + 7, cy=(148.3, 80.0), **WIDE),
    "dense": dict(n=190 * 120),
    "narrow_12_nodes": dict(n=190 * 40, smin=0.62, smax=0.8, half=5),
    "steep": dict(n=190 * 40, cy=(48.3, 44.0)),
    "flat_on_half_integer": dict(n=190 * 40, cy=(47.5,)),
    "many_grid_lines": dict(n=190 * 40, grid=31, cy=(40.3, 20.0)),
    "off_edges": dict(n=240 * 40, xh=120.0, cy=(2.2, 1.4, 0.8)),
    "ragged_f64_spectra": dict(n=126 * 40, nx=129, ny=33, cy=(16.4, 3.0), xh=63.0, dtype=np.float64, traces=1),
}


@pytest.mark.parametrize("prec", list(BOUNDS))
@pytest.mark.parametrize("name", list(CASES))
def test_frames_against_the_oracle(name, prec):
    from tests import gpu_util
    sc = _scene(**CASES[name])
    rq = Request(rv_mps=700.0, flux_scale=1.7, precision=prec)
    print(f"case {name} {prec}", flush=True)
    g, o = gpu_util.render(sc, rq), oracle.render(sc, rq)
    assert metrics.max_rel_err(g, o) < BOUNDS[prec]


@pytest.mark.parametrize("prec", list(BOUNDS))
def test_mixed_batch_equals_single_frames(prec):
    """One batch of frames with 10 nodes, 12 nodes and none (FP64 output)."""
    from tests import gpu_util
    scs = [_scene(n=8000), _scene(n=9000, smin=0.62, smax=0.8, half=5), _scene(n=5000, nx=129, ny=33, xh=60.0)]
    scs[2].out_dtype = "f64"
    c = gpu_util.ctx()
    lds = [gpu_util.P.Loaded(c, sc) for sc in scs]
    rqs = [Request(rv_mps=3.0 * i, flux_scale=1.0 + i, precision=prec) for i in range(3)]
    print(f"mixed batch {prec}", flush=True)
    outs = gpu_util.render_batch(scs, rqs, lds)
    again = gpu_util.render_batch(scs[::-1], rqs[::-1], lds[::-1])[::-1]
    for sc, rq, ld, o, a in zip(scs, rqs, lds, outs, again):
        single = gpu_util.render(sc, rq, loaded=ld)
        assert np.array_equal(o, single) and np.array_equal(a, single)
        ld.free()
