"""A spectrum with one NaN or infinite sample.  An explicit fiber image keeps it inside its own window; a separable
frame inside the window's columns, in the rows of the 16-row blocks its window reaches (the products are taken
block by block).  Elsewhere the frame is the one without it, bit by bit, and an infinity shows as one where its
weight is not zero."""
import numpy as np
import pytest

from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu

V = {"nan": np.nan, "inf": np.inf, "minus_inf": -np.inf}


def _frames(psf, n, value, nx, ny, dtype=np.float32, where=None):
    from tests import gpu_util
    rng = np.random.default_rng(4)
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2 + 0.3 * q, 0.47 * nx, 0.3], [45.3 + 24.0 * q, 6.0], 1.0, q)
           for q in range((ny - 90) // 24)]
    spec = [(1e4 * rng.uniform(0.5, 1.5, n)).astype(dtype) for _ in trs]
    sc = Scene("non_finite", nx, ny, trs, psf, spec, "f32")
    clean = gpu_util.render(sc, Request())
    tr, k = trs[len(trs) // 2], n // 2 + 3 if where is None else where
    spec[tr.slot] = spec[tr.slot].copy()
    spec[tr.slot][k] = value
    t = (2 * k + 1) / n - 1.0
    x, y = np.polynomial.polynomial.polyval(t, tr.cx), np.polynomial.polynomial.polyval(t, tr.cy)
    return clean, gpu_util.render(sc, Request()), int(np.floor(x + 0.5)), int(np.floor(y + 0.5))


@pytest.mark.parametrize("value", list(V))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_fiber_image(value, dtype):
    rng = np.random.default_rng(1)
    psf = Psf(kind="sfi", gx=3, gy=3, half_width=4, sigma_xy=rng.uniform(0.9, 1.3, (3, 3, 2)).astype(np.float32),
              fiber_radius=1.5, fiber_shape="disc", subpix=3)
    for where in (None, 0, 63, 64):  # also the first and the last image of a block of 64
        print(f"case fiber image {value} {where}", flush=True)
        clean, f, ax, ay = _frames(psf, 400, V[value], 190, 140, dtype, where)
        inside = np.zeros(f.shape, bool)
        inside[ay - 4:ay + 5, max(ax - 4, 0):ax + 5] = True
        assert np.array_equal(f[~inside], clean[~inside])
        if value == "nan":
            assert np.isnan(f[inside]).all()
        else:
            assert (f[inside] == V[value]).all()


@pytest.mark.parametrize("value", list(V))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_separable(value, dtype):
    rng = np.random.default_rng(2)
    psf = Psf(kind="separable", gx=3, gy=3, half_width=5, sigma_xy=rng.uniform(1.0, 1.3, (3, 3, 2)).astype(np.float32))
    print(f"case separable {value}", flush=True)
    clean, f, ax, ay = _frames(psf, 1200 * 60, V[value], 1300, 1300, dtype)
    near = np.zeros(f.shape, bool)
    near[(ay - 5) // 16 * 16:((ay + 5) // 16 + 1) * 16, ax - 5:ax + 6] = True
    assert np.array_equal(f[~near], clean[~near])
    inside = f[ay - 5:ay + 6, ax - 5:ax + 6]
    assert np.isnan(inside).all() if value == "nan" else (inside == V[value]).all()
