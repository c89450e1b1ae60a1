"""CCF launches past the limits of one: more velocities than a slice of the partial sums (4096), more traces than
the grid's second dimension holds (65535), sharing one template or each with its own."""
import numpy as np
import pytest

import oracle
from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv", [4096, 4097, 4096 + 700])
def test_velocities_past_a_slice_equal_the_oracle(nv):
    from paper_2008_05858_amd import Loaded
    from tests import gpu_util
    from tests.test_gpu_ccf_paths import _scene
    from tests.test_gpu_loop import gpu_ccf
    sc, dv = _scene(nx=150, n=6000), 2.5
    print(f"case velocities {nv}", flush=True)
    Ex, L = oracle.extract(sc, oracle.render(sc, Request(rv_mps=700.0)), 4.5)
    Co, rvo = oracle.ccf(sc, Ex, L, -0.5 * nv * dv, dv, nv)
    ld = Loaded(gpu_util.ctx(), sc)
    Cg, rvg = gpu_ccf(ld, sc, Ex, L, -0.5 * nv * dv, dv, nv)
    ld.free()
    assert np.max(np.abs(Cg - Co)) <= 1e-9 * np.abs(Co).max()
    assert abs(rvg - rvo) <= 1e-3 * dv


@pytest.mark.parametrize("slots", [1, 66_000])
def test_more_traces_than_a_grid_holds(slots):
    """The rows of some of 66,000 traces are those of a format of these traces alone, bit by bit."""
    from paper_2008_05858_amd import Loaded
    from tests import gpu_util
    from tests.test_gpu_loop import gpu_ccf
    ntr, nx, n, nv = 66_000, 40, 300, 21
    rng = np.random.default_rng(7)
    base = 1.0 + rng.random(n)
    spec = [base] if slots == 1 else [base * f for f in 1.0 + rng.random(ntr)]

    def scene(which):
        trs = [Trace(0, 0, int(q), 600.0, 601.0, n, [19.5, 19.0], [5.0], 1.0, 0 if slots == 1 else i)
               for i, q in enumerate(which)]
        return Scene("many", nx, 10, trs, Psf(kind="erf", sigma=1.0, half_width=3),
                     spec if slots == 1 else [spec[q] for q in which], "f32")

    Ex = rng.random((ntr, nx))
    L = np.broadcast_to(600.0 + (np.arange(nx + 1) - 1.0) / 38.0, (ntr, nx + 1)).copy()
    some = np.concatenate([np.arange(3), np.arange(65530, 65542), np.arange(ntr - 3, ntr)])
    out = []
    for which in (np.arange(ntr), some):
        print(f"case traces {len(which)} slots {slots}", flush=True)
        sc = scene(which)
        ld = Loaded(gpu_util.ctx(), sc)
        out.append(gpu_ccf(ld, sc, Ex[which], L[which], -3000.0, 300.0, nv, smooth_px=0.4)[0])
        ld.free()
    assert np.abs(out[0]).max() > 0 and np.array_equal(out[0][some], out[1])
    assert np.count_nonzero(np.abs(out[0]).max(1) == 0) == 0
