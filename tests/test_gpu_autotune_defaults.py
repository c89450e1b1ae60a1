"""What the autotuner tries: a shape's own default unit length is one of the candidates (3 tiles for frames of 6144
to 16383 tiles, each frame's own where they differ), and launches that have one width only are not timed three
times."""
import numpy as np
import pytest

from workloads import Psf, Request, Scene, Trace, scene
from workloads.synth import elliptical_gaussian_tables

pytestmark = pytest.mark.gpu


def _table(nx=3600, ny=3600):
    """65 x 113 tiles: units of 3 by default."""
    n = 4000
    trs = [Trace(0, 0, q, 600.0, 603.0, n, [nx / 2, 0.47 * nx], [300.0 + 500.0 * q, 20.0], 1.0, q) for q in range(6)]
    tab = elliptical_gaussian_tables(np.random.default_rng(1), 3, 3, 32, 32, 4)
    return Scene("tune", nx, ny, trs, Psf(kind="table", gx=3, gy=3, kw=32, kh=32, os=4, tables=tab),
                 [np.full(n, 5.0, np.float32)] * 6, "f32")


def _tune(scs):
    import paper_2008_05858_amd as P
    from paper_2008_05858_amd import e2e as E
    from tests import gpu_util as gu
    ctx = E.e2e_create(0, 0)
    try:
        lds = [P.Loaded(ctx, sc) for sc in scs]
        reqs, keep = [], []
        for sc, ld in zip(scs, lds):
            specs, sdt = gu.device_spectra(sc)
            out, odt = gu.out_tensor(sc)
            r, k = gu.request_for(ld, sc, specs, sdt, out, odt, Request(rv_mps=3.0))
            reqs.append(r)
            keep.append((specs, out, k))
        rep = E.e2e_autotune(ctx, reqs)
        cands = [(rep.cand_chunk[i], rep.cand_resident[i]) for i in range(rep.n_candidates)]
        print("candidates", cands, "kept", rep.chunk, rep.resident, flush=True)
        outs = gu.render_batch(scs, [Request(rv_mps=3.0)] * len(scs), lds, context=ctx)
        for sc, ld, o in zip(scs, lds, outs):
            assert np.array_equal(o, gu.render(sc, Request(rv_mps=3.0), loaded=ld, context=ctx))
        assert (rep.chunk, rep.resident) in cands
        return cands
    finally:
        E.e2e_destroy(ctx)


def test_a_frame_of_three_tile_units():
    print("case tune one", flush=True)
    assert sorted(c for c, _ in _tune([_table()])) == [2, 3, 4, 8, 16]


def test_batches():
    print("case tune equal", flush=True)
    assert sorted(_tune([_table(), _table()])) == [(c, r) for c in (2, 3, 4, 8, 16) for r in (1, 2, 3)]
    print("case tune unequal", flush=True)
    sc = scene("mini_table")
    assert sorted(_tune([_table(), sc])) == [(c, r) for c in (0, 2, 4, 8, 16) for r in (1, 2, 3)]


def test_a_kind_whose_launches_have_one_width():
    print("case tune separable", flush=True)
    rng = np.random.default_rng(2)
    sc = _table(600, 500)
    sc.psf = Psf(kind="separable", gx=3, gy=3, half_width=5, sigma_xy=rng.uniform(1.0, 1.4, (3, 3, 2)).astype(np.float32))
    assert len(_tune([sc, sc])) == 1
