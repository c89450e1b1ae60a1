"""Separable FP32 frames with more short traces in one 64 x 32 tile than a tile's list holds (512), none of them in
more than a few 16 x 16 tiles: rendered per sample under the FP64 and FP32 precisions, refused under the hi/lo
ones, whose tile is the large one."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace, metrics

pytestmark = pytest.mark.gpu

BOUNDS = {"f64": 1e-6, "f32": 4e-6}  # the requirement; the fitted FP32 tails


def _scene(places, n=60, per=70, half=2):
    """n samples over 6 px; none on a half-integer, where its window would be a matter of rounding."""
    rng = np.random.default_rng(9)
    trs = [Trace(0, 0, q, 600.0, 600.2, n, [x + 0.0317 + 0.001 * q, 3.0], [y + 0.0171 + 0.002 * q, 0.1], 1.0, q % per)
           for q, (x, y) in enumerate(places)]
    psf = Psf(kind="separable", gx=2, gy=2, half_width=half, sigma_xy=rng.uniform(0.9, 1.2, (2, 2, 2)).astype(np.float32))
    return Scene("crowded", 1536, 1536, trs, psf, [(1e4 * rng.uniform(0.2, 1.5, n)).astype(np.float32) for _ in range(per)],
                 "f32")


def _crowd(n=60):
    """700 traces: 350 around x = 650 and as many around x = 690, all of one tile (columns 640 .. 703)."""
    return _scene([(650.0, 655.0)] * 350 + [(690.0, 655.0)] * 350, n)


@pytest.mark.parametrize("prec", list(BOUNDS))
def test_crowded_tile(prec):
    from tests import gpu_util
    sc, rq = _crowd(), Request(rv_mps=0.0, precision=prec)
    print(f"case crowded {prec}", flush=True)
    g, o = gpu_util.render(sc, rq), oracle.render(sc, rq)
    assert metrics.max_rel_err(g, o) < BOUNDS[prec]
    ld = gpu_util.P.Loaded(gpu_util.ctx(), sc)
    assert all(np.array_equal(g, b) for b in gpu_util.render_batch([sc] * 2, [rq] * 2, [ld] * 2))
    ld.free()


def test_crowded_tile_dense_enough_for_nodes_under_fp32():
    """15 samples a pixel.  FP32 sums of 350 x 90 samples: 3e4 roundings of 3e-8 at random are 5e-6, four times
    that the bound."""
    from tests import gpu_util
    sc, rq = _crowd(90), Request(rv_mps=0.0, precision="f32")
    print("case crowded f32, 15 a pixel", flush=True)
    assert metrics.max_rel_err(gpu_util.render(sc, rq), oracle.render(sc, rq)) < 2e-5


def test_crowded_tile_of_the_hilo_kernels_is_refused():
    from tests import gpu_util
    from paper_2008_05858_amd import e2e as E
    print("case crowded f16_hilo", flush=True)
    with pytest.raises(E.E2EError, match="too many traces"):
        gpu_util.render(_crowd(), Request(precision="f16_hilo"))
