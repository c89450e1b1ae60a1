"""The partial sums of split tiles are given back when an allocation fails, also one of the very call that was
going to use them: its kernels then have to do without.  The library's host code on a stand-in runtime
(fake_hip.cpp) that refuses one allocation after another; no kernel may be given memory that was freed."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # ahead of the library's own runtime
for f in ("refused", "units", "bad", "mallocs"):
    getattr(fake, "fake_" + f).restype = C.c_long
fake.fake_fail_at.argtypes = [C.c_long]
import numpy as np
import paper_2008_05858_amd as P
from paper_2008_05858_amd import e2e as E
from workloads import Psf, Scene, Trace
n, host = 600, sys.argv[2] == "host"
tr = [Trace(0, 0, 0, 600.0, 603.0, n, [32.0, 30.0], [16.0], 1.0, 0)]
sc = Scene("kept", 64, 32, tr, Psf(kind="erf", sigma=1.2, half_width=5), [np.ones(n)], "f64")

def render(ctx, ld, at):
    spec, out = np.ones(n), np.zeros((32, 64))
    r, keep = P.make_req(ld, [spec.ctypes.data], E.E2E_F64, out.ctypes.data, E.E2E_F64,
                         spectra_on_device=not host, out_on_device=not host, rv_mps=0.0, flux_scale=1.0, seed=0,
                         frame_index=0, poisson=False, precision="f64")
    before = fake.fake_units(), fake.fake_mallocs(), fake.fake_refused()
    fake.fake_fail_at(at)
    E.e2e_render(ctx, r)
    fake.fake_fail_at(-1)
    return fake.fake_units() - before[0], fake.fake_mallocs() - before[1], fake.fake_refused() - before[2]

def kept():
    ctx = E.e2e_create(0, 1 << 30)
    ld = P.Loaded(ctx, sc)
    u, _, _ = render(ctx, ld, -1)
    assert u == 2, u                                # split tiles ran: units and their sum
    return ctx, ld

ctx, ld = kept()
u, calls, _ = render(ctx, ld, -1)
assert u == 2 and calls == (2 if host else 0), (u, calls)
E.e2e_destroy(ctx)
for at in range(calls):
    ctx, ld = kept()
    u, _, refused = render(ctx, ld, at)
    print("refused allocation", at, "split launches", u, "freed", fake.fake_bad(), flush=True)
    assert refused == 1 and u == 0                  # accepted all the same, without the sums
    u, _, _ = render(ctx, ld, -1)
    assert u == 2                                   # and with them again by the next call
    E.e2e_destroy(ctx)
assert fake.fake_bad() == 0, fake.fake_bad()
print("done")
"""


@pytest.mark.parametrize("where", ["device", "host"])
def test_refused_allocations(where, tmp_path):
    so = str(tmp_path / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.cpp")], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, so, where], cwd=os.path.dirname(HERE), timeout=100,
                       capture_output=True, text=True)
    assert r.returncode == 0 and "done" in r.stdout, r.stdout + r.stderr
