"""Detector stage where its shortcuts could decide wrongly: a bias that cancels nearly all of a pixel's charge (the
roundings of the charge's quotient are then much larger than those of the sum)."""
import numpy as np
import pytest

from tests.test_gpu_detector import _gpu_detector, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,gain", [(1e13, 1.1), (3e11, 0.7), (-4e12, 1.3)])
def test_a_bias_that_cancels_the_charge(base, gain):
    """Without shot noise, read noise of 1e-6 electrons: divide, add and floor only, bit for bit."""
    rng = np.random.default_rng(3)
    F = base + rng.uniform(0.0, 4e4, (217, 301))
    kw = dict(shot_noise=False, ron_e=1e-6, gain=gain, bias=-np.floor(base / gain), seed=5)
    print(f"case detector bias {base} {gain}", flush=True)
    g, o = _gpu_detector(F, None, kw), _oracle(F, None, kw)
    assert o.max() > 20000 and np.array_equal(g, o), np.count_nonzero(g != o)
