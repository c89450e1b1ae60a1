"""Which kernel renders a frame, by the launch names of the profile, and the accuracy of the column nodes under every
precision: their frames keep 3e-7 of the peak (1.7e-7 measured at the most), whatever the per-sample kernel of that
precision leaves."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_sep_fit import CASES, _scene
from workloads import Psf, Request, Scene, Trace, metrics

pytestmark = pytest.mark.gpu

KERNELS = ("render_sep_fit", "render_sep_units", "render_sfi_terms")


class _Launches:
    """Launches by kernel name while in scope."""

    def __enter__(self):
        from tests import gpu_util
        self.E, self.ctx = gpu_util.E, gpu_util.ctx()
        self.E.e2e_reset_kernel_time(self.ctx)
        self.E.e2e_set_profiling(self.ctx, 1)
        return self

    def __exit__(self, *exc):
        self.n = {k: self.E.e2e_kernel_time(self.ctx, k)[0] for k in (*KERNELS, "render_sep", "render_sep_mfma", "render_sfi")}
        self.E.e2e_set_profiling(self.ctx, 0)
        return False


def _dense(kw, prec):
    """The case with enough samples for the nodes: 9500 tiles times samples a pixel under FP64."""
    kw = dict(kw)
    tiles = -(-kw.get("nx", 203) // 64) * -(-kw.get("ny", 97) // 32)
    span = 2.0 * kw.get("xh", 95.0)
    if prec == "f64" and not kw.get("short"):
        kw["n"] = max(kw["n"], int(1.02 * span * max(9500.0 / tiles, 6.0)) + 3)
    elif prec == "f64":  # the mean over both traces, one of them of a sample or two
        kw["n"] = int(2.1 * span * 9500.0 / tiles)
    elif kw.get("short"):
        kw["n"] = int(2.1 * span * 36)
    return kw


@pytest.mark.parametrize("prec", ["f64", "f32", "f16_hilo", "bf16_hilo"])
@pytest.mark.parametrize("name", list(CASES))
def test_column_nodes(name, prec):
    from tests import gpu_util
    sc = _scene(**_dense(CASES[name], prec))
    rq = Request(rv_mps=700.0, flux_scale=1.7, precision=prec)
    print(f"case nodes {name} {prec}", flush=True)
    with _Launches() as seen:
        g = gpu_util.render(sc, rq)
    asked = "render_sep" if prec in ("f64", "f32") else "render_sep_mfma"
    assert seen.n["render_sep_fit"] == 1 and seen.n[asked] == 1 and seen.n["render_sep_units"] == 0
    assert metrics.max_rel_err(g, oracle.render(sc, rq)) < 3e-7


@pytest.mark.parametrize("prec", ["f64", "f16_hilo"])
def test_mixed_batch_of_ten_nodes_twelve_and_none(prec):
    from tests import gpu_util
    n = 190 * 620
    scs = [_scene(n=n), _scene(n=n, smin=0.62, smax=0.8, half=5), _scene(n=5000, nx=129, ny=33, xh=60.0), _scene(n=n)]
    scs[2].out_dtype = "f64"
    lds = [gpu_util.P.Loaded(gpu_util.ctx(), sc) for sc in scs]
    rqs = [Request(rv_mps=3.0 * i, flux_scale=1.0 + i, precision=prec) for i in range(4)]
    print(f"case nodes mixed {prec}", flush=True)
    with _Launches() as seen:
        outs = gpu_util.render_batch(scs, rqs, lds)
    assert seen.n["render_sep_fit"] == 2 and seen.n["render_sep" if prec == "f64" else "render_sep_mfma"] == 3
    for sc, rq, ld, o in zip(scs, rqs, lds, outs):
        assert np.array_equal(o, gpu_util.render(sc, rq, loaded=ld))
        ld.free()


def test_frames_that_keep_the_per_sample_kernels():
    from tests import gpu_util
    print("case per sample", flush=True)
    for kw, prec, out, names in ((dict(n=190 * 40), "f64", "f32", ("render_sep_units",)),   # too few tiles
                                 (dict(n=190 * 700), "f64", "f64", ("render_sep_units",)),  # FP64 frame
                                 (dict(n=190 * 20), "f32", "f32", ()), (dict(n=190 * 10), "f16_hilo", "f32", ()),
                                 (dict(n=190 * 700, smin=0.4, smax=0.6), "f64", "f32", ("render_sep_units",))):
        sc = _scene(**kw)
        sc.out_dtype = out
        with _Launches() as seen:
            gpu_util.render(sc, Request(precision=prec))
        assert {k for k in KERNELS if seen.n[k]} == set(names), (kw, prec, out)


def test_fiber_images():
    from tests import gpu_util
    print("case fiber images", flush=True)
    for smin, out, n in ((0.8, "f32", 1), (0.5, "f32", 0), (0.8, "f64", 0)):
        psf = Psf(kind="sfi", gx=2, gy=2, half_width=4, sigma_xy=np.full((2, 2, 2), smin, np.float32), fiber_radius=1.0,
                  fiber_shape="disc", subpix=2)
        tr = [Trace(0, 0, 0, 600.0, 603.0, 90, [45.0, 30.0], [24.3, 6.0], 1.0, 0)]
        with _Launches() as seen:
            gpu_util.render(Scene("sfi", 90, 50, tr, psf, [np.ones(90, np.float32)], out))
        assert seen.n["render_sfi_terms"] == n and seen.n["render_sfi"] == 1


def test_many_traces_far_apart_keep_the_column_nodes():
    """900 traces of a 1536^2 frame, at most 18 in a tile; 700 in one tile do not."""
    from tests import gpu_util
    from tests.test_gpu_crowded_tiles import _crowd, _scene as short_traces
    print("case many traces", flush=True)
    apart = short_traces([(20.0 + 50.0 * (q % 30), 20.0 + 50.0 * (q // 30)) for q in range(900)], n=90)
    for sc, n in ((apart, 1), (_crowd(90), 0)):
        for prec in ("f64", "f32"):
            with _Launches() as seen:
                gpu_util.render(sc, Request(precision=prec))
            assert seen.n["render_sep_fit"] == n and seen.n["render_sep"] == 1
