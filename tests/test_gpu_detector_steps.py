"""Detector stage where its shortcuts could decide wrongly: a bias that cancels nearly all of a pixel's charge (the
roundings of the charge's quotient are then much larger than those of the sum), and frames of more tile rows than
one layer of the grid holds."""
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


@pytest.mark.parametrize("ny", [32768 * 48 - 1, 32768 * 48 + 1, 1_600_000])
def test_more_rows_than_a_layer_of_the_grid(ny):
    """A column of pixels: the read-out without cross-talk at unit gain is the Poisson draw of the same stream."""
    import torch
    from paper_2008_05858_amd import e2e as E
    from tests import gpu_util
    g = torch.Generator(device="cuda").manual_seed(ny)
    f = 40.0 * torch.rand((ny,), generator=g, device="cuda")
    print(f"case detector rows {ny}", flush=True)
    adu = _gpu_detector(f.cpu().numpy().reshape(ny, 1), None, dict(shot_noise=True, seed=8, frame=2))
    E.e2e_noise_poisson(gpu_util.ctx(), f.data_ptr(), E.E2E_F32, ny, 8, 2, 1)
    assert np.array_equal(adu[:, 0], f.cpu().numpy().astype(np.uint16))
