"""CPU: the fitted Mills ratio of the explicit-SFI term kernel (mills() in
csrc/k_sfi_terms.hip), its coefficients read from the source, against scipy:
relative error below 1.2e-9 on [0, 9], and bounded beyond, where the Gaussian
it multiplies is below 3e-18."""
import os
import re

import numpy as np
from scipy.special import erfcx

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2008_05858_amd", "csrc", "k_sfi_terms.hip")


def test_fitted_mills_ratio():
    src = open(SRC).read()
    body = src[src.index("double mills(double z)"):]
    body = body[:body.index("\n}\n")]
    num = r"(-?\d+\.\d+e[+-]\d+)"
    c = [float(re.search(r"double p = " + num, body).group(1))]
    c += [float(v) for v in re.findall(r"fma\(p, t, " + num + r"\)", body)]
    a = float(re.search(r"fma\((\d+\.\d+), z, 1\.0\)", body).group(1))
    assert len(c) == 11
    z = np.linspace(0.0, 9.0, 90001)
    ref = np.sqrt(np.pi / 2) * erfcx(z / np.sqrt(2.0))
    assert np.max(np.abs(np.polyval(c, 1.0 / (1.0 + a * z)) / ref - 1.0)) < 1.2e-9
    far = np.linspace(9.0, 40.0, 10001)
    assert np.max(np.abs(np.polyval(c, 1.0 / (1.0 + a * far)))) < 1.0
