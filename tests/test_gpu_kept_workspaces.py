"""Workspaces that a context keeps between calls (the CCF's, the partial sums of split tiles) stay within its memory
budget, and give way to loads and renders that need their room: what fits the budget without them is accepted.
Device memory as the driver reports it; 24 MB of slack for its own allocations (2 MB pages, code, streams)."""
import numpy as np
import pytest

from workloads import Psf, Request, Scene, Trace

pytestmark = pytest.mark.gpu

MB = 1 << 20
SLACK = 24 * MB


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _erf(nx=1024, ny=1024):
    """4096 tiles: 96 MB of partial sums."""
    rng = np.random.default_rng(6)
    n = 20 * nx
    tr = [Trace(0, 0, 0, 600.0, 603.0, n, [nx / 2, 0.47 * nx, 0.3], [ny / 2, 20.0, 1.0], 1.0, 0)]
    return Scene("kept", nx, ny, tr, Psf(kind="erf", sigma=1.2, half_width=5), [1e4 * rng.random(n)], "f32")


def _ccf_call(ctx):
    """A CCF of 22 templates of 1e6 samples: 176 MB of workspace."""
    import torch
    from paper_2008_05858_amd import Loaded
    from paper_2008_05858_amd import e2e as E
    n, ntr, nx, nv = 1_000_000, 22, 512, 11
    trs = [Trace(0, 0, q, 600.0 + q, 601.0 + q, n, [255.5, 250.0], [5.0 + q], 1.0, q) for q in range(ntr)]
    ld = Loaded(ctx, Scene("ccf", nx, 64, trs, Psf(kind="erf", sigma=1.0, half_width=3), [], "f32"))
    g = torch.Generator(device="cuda").manual_seed(1)
    t = torch.rand((ntr, n), generator=g, device="cuda")
    flux = torch.rand((ntr, nx), generator=g, device="cuda", dtype=torch.float64)
    x = (torch.arange(nx + 1, device="cuda", dtype=torch.float64) - 6.0) / 500.0
    edges = 600.0 + torch.arange(ntr, device="cuda", dtype=torch.float64)[:, None] + x[None]
    out = torch.zeros((ntr, nv), device="cuda", dtype=torch.float64)
    r = E.e2e_ccf_req()
    ptr = (E.C.c_void_p * ntr)(*[row.data_ptr() for row in t])
    r.flux, r.edges, r.ccf_out = flux.data_ptr(), edges.data_ptr(), out.data_ptr()
    r.templates = E.C.cast(ptr, E.C.POINTER(E.C.c_void_p))
    r.n_templates, r.template_dtype, r.on_device = ntr, E.E2E_F32, 1
    r.n_v, r.dv_mps, r.v0_mps, r.smooth_px = nv, 100.0, -500.0, 0.05
    torch.cuda.synchronize()
    return ld, lambda: (E.e2e_ccf(ctx, ld.fmt, r), out.cpu().numpy())[1], (t, flux, edges, out, ptr)


def test_ccf_workspace_within_the_budget():
    from paper_2008_05858_amd import e2e as E
    res = []
    for budget in (64 * MB, 400 * MB):
        print(f"case ccf budget {budget // MB} MB", flush=True)
        ctx = E.e2e_create(0, budget)
        try:
            ld, call, keep = _ccf_call(ctx)
            before = _free()
            res.append(call())
            used = before - _free()
            assert used <= (SLACK if budget < 100 * MB else 180 * MB + SLACK), used
            assert np.array_equal(res[-1], call())
            ld.free()
        finally:
            E.e2e_destroy(ctx)
    assert np.abs(res[0]).max() > 0 and np.array_equal(res[0], res[1])


def test_split_tiles_of_several_streams_within_the_budget():
    """Three streams' partial sums take 289 MB; two of them and the frames fit 220 MB.  The same bits on each."""
    import torch
    from paper_2008_05858_amd import Loaded
    from paper_2008_05858_amd import e2e as E
    from tests import gpu_util
    sc = _erf()
    ctx = E.e2e_create(0, 220 * MB)
    try:
        ld = Loaded(ctx, sc)
        specs, sdt = gpu_util.device_spectra(sc)
        outs = [gpu_util.out_tensor(sc)[0] for _ in range(3)]
        streams = [torch.cuda.Stream() for _ in range(3)]
        before = _free()
        for o, s in zip(outs, streams):
            print("case stream", flush=True)
            r, keep = gpu_util.request_for(ld, sc, specs, sdt, o, E.E2E_F32, Request(rv_mps=5.0), stream=s.cuda_stream)
            torch.cuda.synchronize()
            E.e2e_render(ctx, r)
        used = before - _free()
        assert used <= 220 * MB + SLACK, used
        f = [o.cpu().numpy() for o in outs]
        assert f[0].max() > 0 and np.array_equal(f[0], f[1]) and np.array_equal(f[0], f[2])
        ld.free()
    finally:
        E.e2e_destroy(ctx)


def test_kept_workspaces_give_way():
    """Within 400 MB: a CCF (176 MB kept) and split tiles (96 MB), then a render of host spectra and a host frame of
    240 MB, and the first two again."""
    from paper_2008_05858_amd import Loaded
    from paper_2008_05858_amd import e2e as E
    from tests import gpu_util
    ctx = E.e2e_create(0, 400 * MB)
    try:
        ld, call, keep = _ccf_call(ctx)
        a = call()
        sc = _erf()
        ls = Loaded(ctx, sc)
        f = gpu_util.render(sc, Request(rv_mps=5.0), loaded=ls, context=ctx)
        before = _free()
        big = Scene("big", 8000, 8000, sc.traces, sc.psf, sc.spectra, "f32")
        lb = Loaded(ctx, big)
        out = np.zeros((8000, 8000), np.float32)
        r, keep2 = gpu_util.P.make_req(lb, [s.ctypes.data for s in sc.spectra], E.E2E_F64, out.ctypes.data, E.E2E_F32,
                                       spectra_on_device=False, out_on_device=False)
        print("case give way", flush=True)
        E.e2e_render(ctx, r)
        assert out.max() > 0 and before - _free() <= 400 * MB
        assert np.array_equal(a, call())
        assert np.array_equal(f, gpu_util.render(sc, Request(rv_mps=5.0), loaded=ls, context=ctx))
        for x in (ld, ls, lb):
            x.free()
    finally:
        E.e2e_destroy(ctx)
