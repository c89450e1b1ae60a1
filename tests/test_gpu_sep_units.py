"""Per-sample FP64 frames of few tiles, whose tiles are summed in units of whole
blocks of samples by workgroups of their own: fewer blocks than units, as
many, one more (two blocks a unit), several traces in a tile, a last block of
one sample, tiles without samples; and the same frame in a batch of more tiles
than take this path, bit by bit.  The bound is the requirement on a frame,
1e-6 of its peak."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics

pytestmark = pytest.mark.gpu


def _scene(kind, per_px, nx=75, ny=41, half=5, traces=1, out="f64", cy=(20.3, 2.0, 1.0), dtype=np.float64):
    rng = np.random.default_rng(11)
    n = int(per_px * 2 * 0.47 * nx)
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.85 * q, 0.47 * nx, 0.3], [cy[0] + 4.0 * q, *cy[1:]], 0.5, q)
           for q in range(traces)]
    spec = [(1e4 * rng.uniform(0.2, 1.5, n)).astype(dtype) for _ in trs]
    psf = Psf(kind="erf", sigma=1.2, half_width=half) if kind == "erf" else Psf(
        kind="separable", gx=3, gy=3, half_width=half,
        sigma_xy=rng.uniform(1.0, 1.4, (3, 3, 2)).astype(np.float32))
    return Scene("sep_units", nx, ny, trs, psf, spec, out)


# a tile column of the middle holds the samples of 16 + 2 half + about 1 pixels
CASES = {
    "one_block": dict(per_px=3.0), "some": dict(per_px=20.0), "as_many_as_units": dict(per_px=57.3),
    "two_a_unit": dict(per_px=61.0), "many_a_unit": dict(per_px=400.0),
    "several_traces": dict(per_px=30.0, traces=4), "few_samples": dict(per_px=0.4, traces=2),
    "off_the_edge": dict(per_px=25.0, cy=(1.0, 3.0)), "f32_out": dict(per_px=33.0, out="f32", dtype=np.float32),
}


@pytest.mark.parametrize("kind", ["erf", "separable"])
@pytest.mark.parametrize("name", list(CASES))
def test_frames_against_the_oracle_and_a_large_batch(name, kind):
    from tests import gpu_util
    kw = dict(CASES[name])
    if kind == "separable" and "out" not in kw:
        kw["out"] = "f64"  # (FP32 frames of dense traces go through column nodes)
    sc = _scene(kind, **kw)
    rq = Request(rv_mps=-700.0, flux_scale=1.7)
    print(f"case {name} {kind}", flush=True)
    ld = gpu_util.P.Loaded(gpu_util.ctx(), sc)
    g, o = gpu_util.render(sc, rq, loaded=ld), oracle.render(sc, rq)
    assert metrics.max_rel_err(g, o) < 1e-6
    # 5 x 3 tiles each: 280 frames are past the limit of 4096 tiles, 3 are not;
    # 1100 are past 16384, where a thread takes two pixels
    for count in (3, 280, 1100) if name == "two_a_unit" else (3, 280):
        outs = gpu_util.render_batch([sc] * count, [rq] * count, [ld] * count)
        assert all(np.array_equal(g, b) for b in outs)
    ld.free()


def test_a_budget_without_room_for_the_units_gives_the_same_bits():
    """15 tiles' partial sums take 15 x 12 x 2 KB, more than this context has."""
    from tests import gpu_util
    from paper_2008_05858_amd import e2e as E
    sc, rq = _scene("erf", 61.0, traces=2), Request(rv_mps=12.0)
    print("case budget", flush=True)
    small = E.e2e_create(0, 200_000)
    try:
        ld = gpu_util.P.Loaded(small, sc)
        a = gpu_util.render(sc, rq, loaded=ld, context=small)
        ld.free()
    finally:
        E.e2e_destroy(small)
    assert np.array_equal(a, gpu_util.render(sc, rq))
