"""Weighted FP32 intensities of the 4 x 256 lattice where the largest weights
belong to many antennas without data: the sums of the others keep their bits,
as with one such antenna (the bound on the 2-norm of the error is derived in
tests/test_gpu_weighted256.py)."""
import numpy as np
import pytest

import oracle as orc
from tests.test_gpu_weighted256 import _run, _volts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("strong", [1500.0, 1e6, 1e20, 1e30])
@pytest.mark.parametrize("dead", [(2, 3), (0, 1, 3)])           # half and three quarters of the antennas
def test_strong_weights_of_dead_antennas(gains, strong, dead):
    rng = np.random.default_rng(7)
    v = _volts(2, 1, 64, 15)
    v[..., list(dead)] = 0
    h = rng.uniform(0.5, 1.3, (256, 4))
    if gains:
        h = h * np.exp(1j * rng.uniform(-np.pi, np.pi, (256, 4)))
    h[:, list(dead)] *= strong
    h = h.astype(np.complex64 if gains else np.float32)
    got = _run(v, h, 16, gains=gains).astype(np.float64)
    ref = orc.beamform_fft(v, 4, 512, 16, taper=h.astype(np.complex128 if gains else np.float64))
    assert np.linalg.norm(got - ref) < 1.7e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("ratio", [2.0 ** -9, 2.0 ** -10, 2.0 ** -10 * 0.999, 2.0 ** -11])
def test_at_the_rule(ratio):
    """Live weights on both sides of 2^-10 of the dead antennas'."""
    rng = np.random.default_rng(9)
    v = _volts(2, 1, 64, 16)
    v[:, :, :, ::2] = 0
    h = rng.uniform(1.0, 1.9, (256, 4)) * ratio
    h[::2] = 1.0
    h[1::2] = np.maximum(h[1::2], ratio)
    h = h.astype(np.float32)
    got = _run(v, h, 16).astype(np.float64)
    ref = orc.beamform_fft(v, 4, 512, 16, taper=h.astype(np.float64))
    assert np.linalg.norm(got - ref) < 1.7e-7 * np.linalg.norm(ref)
