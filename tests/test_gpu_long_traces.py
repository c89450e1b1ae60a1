"""Traces of more than 2^30 samples.  Under constant photons a frame does not depend on the sampling (the
samples' sum is the midpoint rule of a smooth integral, at 2500 samples a pixel within 1e-8 of it), so the
frame of so many samples is the one of a thousandth as many.  Both frames keep the requirement of 1e-6 of the
peak, and each is an FP32 frame of ordinary rounding (1e-7): within 5e-7 of each other."""
import numpy as np
import pytest

from workloads import Psf

pytestmark = pytest.mark.gpu


def _frame(psf, n, nx=512, ny=64):
    import torch
    from tests import gpu_util
    from workloads import Scene, Trace
    tr = [Trace(0, 0, 0, 600.0, 603.0, n, [nx / 2, 0.47 * nx, 0.3], [ny / 2 + 0.3, 3.0, 1.0], 1.0, 0)]
    sc = Scene("long", nx, ny, tr, psf, [np.zeros(0, np.float32)], "f32")
    ld = gpu_util.P.Loaded(gpu_util.ctx(), sc)
    spec = torch.full((n,), 1.0, dtype=torch.float32, device="cuda")
    out, odt = gpu_util.out_tensor(sc)
    r, keep = gpu_util.request_for(ld, sc, [spec], gpu_util.E.E2E_F32, out, odt, rv_mps=300.0, flux_scale=1e9 / n)
    torch.cuda.synchronize()
    gpu_util.E.e2e_render(gpu_util.ctx(), r)
    f = out.cpu().numpy().astype(np.float64)
    ld.free()
    del spec
    torch.cuda.empty_cache()
    return f


def _table():
    """Nine round maps, each with its own width."""
    maps = np.empty((3, 3, 32, 32), np.float32)
    u = (np.arange(32) - 15.5) / 4.0
    for q in range(9):
        g = np.exp(-0.5 * (u / (1.0 + 0.05 * q)) ** 2)
        maps[q // 3, q % 3] = np.outer(g, g) / g.sum() ** 2
    return Psf(kind="table", gx=3, gy=3, kw=32, kh=32, tables=maps)


@pytest.mark.parametrize("kind", ["separable", "table"])
@pytest.mark.parametrize("n", [2**30 + 12_345_678, 2**31 - 2])
def test_the_frame_of_a_thousandth_as_many_samples(kind, n):
    rng = np.random.default_rng(2)
    psf = _table() if kind == "table" else Psf(
        kind="separable", gx=3, gy=3, half_width=6, sigma_xy=rng.uniform(1.0, 1.4, (3, 3, 2)).astype(np.float32))
    print(f"case long {kind} {n}", flush=True)
    a, b = _frame(psf, n), _frame(psf, n // 1000)
    assert b.max() > 0 and abs(a.sum() / b.sum() - 1.0) < 1e-6
    assert np.max(np.abs(a - b)) < 5e-7 * b.max()
