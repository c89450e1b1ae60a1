"""Index arithmetic of the kernels on traces of up to 2^31 - 2 samples, compiled
for the host: no result may wrap in 32 bits."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2008_05858_amd", "csrc")
MOST = 2**31 - 2  # samples of a trace


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("sample_index")
    src = d / "s.cpp"
    src.write_text("""
#define __host__
#define __device__
#include "sample_index.h"
extern "C" int room(int n, int g, int place) { return e2e::group_room(n, g, place); }
extern "C" int group(int room, int off) { return e2e::group_inside(room, off); }
extern "C" int value(int room, int g, int off, int e) { return e2e::value_inside(room, g, off, e); }
extern "C" double node(int ks, int ke, double tau) { return e2e::node_sample(ks, ke, tau); }
""")
    so = d / "s.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    d = ctypes.CDLL(str(so))
    d.node.restype = ctypes.c_double
    d.node.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_double]
    for f, k in ((d.room, 3), (d.group, 2), (d.value, 4)):
        f.argtypes = [ctypes.c_int] * k
    return d


@pytest.mark.parametrize("ks,ke", [(0, 1), (5, 90), (2**29, 2**29 + 7), (2**30 - 3, 2**30 + 4), (2**30 + 5, 2**30 + 900),
                                   (MOST - 90, MOST), (0, MOST)])
def test_node_places(lib, ks, ke):
    """-1 and 1 are the column's first and last sample, 0 the middle between them."""
    assert lib.node(ks, ke, -1.0) == ks
    assert lib.node(ks, ke, 1.0) == ke - 1
    assert lib.node(ks, ke, 0.0) == (ks + ke - 1) / 2


@pytest.mark.parametrize("n", [1, 3, 4, 1000, MOST - 60_000, MOST])
def test_groups_inside_the_spectrum(lib, n):
    """A column's first sample (up to n: none), a lane's chunk of a block and up to n - 1 samples read ahead:
    groups and values count as inside exactly where their indices are."""
    near = sorted({q for q in (0, 1, 2, n // 2, n - 60_000, n - 19, n - 5, n - 4, n - 1, n) if 0 <= q <= n})
    for g in (2, 4):
        for first in near:
            for chunk in range(4):
                room = lib.room(n, g, first) - g * chunk
                for off in [q for q in near if q < n]:
                    k = first + g * chunk + off
                    assert bool(lib.group(room, off)) == (k + g <= n), (g, first, chunk, off)
                    for e in range(g):
                        assert bool(lib.value(room, g, off, e)) == (k + e < n), (g, first, chunk, off, e)
                        if k + e < n:  # the index taken from the spectrum's last g values
                            assert (n - g) + (off - room) + e == k + e and abs(off - room) < 2**31
