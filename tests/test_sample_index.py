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
extern "C" double node(int ks, int ke, double tau) { return e2e::node_sample(ks, ke, tau); }
""")
    so = d / "s.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    d = ctypes.CDLL(str(so))
    d.node.restype = ctypes.c_double
    d.node.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_double]
    return d


@pytest.mark.parametrize("ks,ke", [(0, 1), (5, 90), (2**29, 2**29 + 7), (2**30 - 3, 2**30 + 4), (2**30 + 5, 2**30 + 900),
                                   (MOST - 90, MOST), (0, MOST)])
def test_node_places(lib, ks, ke):
    """-1 and 1 are the column's first and last sample, 0 the middle between them."""
    assert lib.node(ks, ke, -1.0) == ks
    assert lib.node(ks, ke, 1.0) == ke - 1
    assert lib.node(ks, ke, 0.0) == (ks + ke - 1) / 2
