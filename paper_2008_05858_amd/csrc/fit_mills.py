"""Coefficients of mills() in k_sfi_terms.hip: the Mills ratio of the normal
distribution,

  M(z) = sqrt(2 pi) Phi(-z) exp(z^2 / 2),  z >= 0,

as a degree-10 polynomial in t = 1 / (1 + 0.35 z), least squares in relative
error on 0 <= z <= 9 (Chebyshev points).  Prints the coefficients (constant
term first) and the largest relative error.  Needs numpy and scipy; run by
hand, not at build time.
"""
import numpy as np
from scipy.special import erfcx

A, DEG, ZMAX = 0.35, 10, 9.0


def mills(z):
    return np.sqrt(np.pi / 2) * erfcx(z / np.sqrt(2.0))


def fit():
    t0 = 1.0 / (1.0 + A * ZMAX)
    x = np.cos(np.pi * (np.arange(400) + 0.5) / 400)
    t = t0 + (1.0 - t0) * (x + 1.0) / 2.0
    w = 1.0 / mills((1.0 / t - 1.0) / A)
    c = np.linalg.lstsq(np.polynomial.chebyshev.chebvander(x, DEG) * w[:, None], np.ones(400), rcond=None)[0]
    return np.polynomial.chebyshev.Chebyshev(c, domain=[t0, 1.0]).convert(kind=np.polynomial.Polynomial).coef


if __name__ == "__main__":
    c = fit()
    print(", ".join(f"{v:.17e}" for v in c))
    z = np.linspace(0.0, ZMAX, 100001)
    got = np.polynomial.polynomial.polyval(1.0 / (1.0 + A * z), c)
    print(f"max relative error: {np.max(np.abs(got / mills(z) - 1.0)):.2e}")
