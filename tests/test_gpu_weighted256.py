"""Weighted FP32 intensities of the 4 x 256 lattice (stage 1 of the N-S
transform on the matrix cores, two FP16 terms per operand) where the split,
the scaling and the pairs of wavefronts can go wrong, against the FP64 oracle.

Tolerance: |B| carries about sqrt(log2 512) + 3 roundings of 2^-24 of its
partial sums' size, whose mean square is the beam's own for noise, so a block
sum of 4 or more |B|^2 is held to the FP32 bar of 1e-5 per beam; the window of
one strong antenna has beams of one size, so it holds there as well."""
import numpy as np
import pytest

import oracle as orc
import synthgen as sg
from tests.helpers import TOL_FP32, rel_err

pytestmark = pytest.mark.gpu


def _run(v, weights, block, pol_sum=False, sel=None, gains=False):
    import torch
    import paper_1710_08591_amd as bf
    t, c, p = v.shape[:3]
    plan = bf.Plan(n_ew=4, n_ns=256, n_pol=p, n_chan=c, block=block, pol_sum=pol_sum, ns_select=sel)
    w = torch.from_numpy(weights).cuda()
    out = bf.beamform_fft(plan, torch.from_numpy(v).cuda(), **({"gains": w} if gains else {"taper": w}))
    out = out.cpu().numpy()
    plan.close()
    return out


def _volts(n_chan, n_pol, n_time, seed):
    return sg.volts(sg.custom_workload(n_ew=4, n_ns=256, n_chan=n_chan, n_pol=n_pol, n_time=n_time, seed=seed, n_src=2,
                                       snr=10.0))


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("n_chan,n_pol,n_blk,block,pol_sum,keep", [
    (1, 1, 1, 4, False, 0),        # one wavefront of a pair
    (3, 1, 3, 20, False, 7),       # an odd count of tasks, a clamp
    (2, 2, 2, 12, True, 512),      # summed polarisations, a permuted clamp of every beam
])
def test_shapes(gains, n_chan, n_pol, n_blk, block, pol_sum, keep):
    rng = np.random.default_rng(block)
    v = _volts(n_chan, n_pol, n_blk * block, block)
    h = rng.uniform(0.2, 1.3, (256, 4)).astype(np.float32)
    if gains:
        h = (h * np.exp(1j * rng.uniform(-np.pi, np.pi, (256, 4)))).astype(np.complex64)
    sel = np.stack([rng.permutation(512)[:keep] for _ in range(n_chan)]).astype(np.int32) if keep else None
    got = _run(v, h, block, pol_sum, sel, gains)
    ref = orc.beamform_fft(v, 4, 512, block, taper=h.astype(np.complex128 if gains else np.float64), ns_select=sel,
                           pol_sum=pol_sum)
    assert got.shape == ref.shape
    assert rel_err(got, ref) < TOL_FP32


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("scale", [1e-15, 3e-3, 1.0, 65504.0, 1e16])
def test_scales(gains, scale):
    """Weights far from 1, of both signs, and one antenna a thousand times the rest."""
    rng = np.random.default_rng(3)
    v = _volts(1, 1, 16, 9)
    h = rng.normal(size=(256, 4))
    if gains:
        h = h + 1j * rng.normal(size=(256, 4))
    h[100, 2] = 1000.0
    h = (h * scale).astype(np.complex64 if gains else np.float32)
    got = _run(v, h, 16, gains=gains)
    ref = orc.beamform_fft(v, 4, 512, 16, taper=h.astype(np.complex128 if gains else np.float64))
    assert rel_err(got, ref) < TOL_FP32


def test_zero_and_infinite_weights():
    v = _volts(1, 1, 16, 4)
    assert not np.any(_run(v, np.zeros((256, 4), np.float32), 16))
    h = np.ones((256, 4), np.float32)
    h[3, 1] = np.inf
    assert not np.any(np.isfinite(_run(v, h, 16)))
    h[3, 1] = np.nan
    assert np.all(np.isnan(_run(v, h, 16)))


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("strong", [1000.0, 3000.0, 1e6, 1e20])
def test_strong_weight_of_a_dead_antenna(gains, strong):
    """The largest weight belongs to an antenna without data: the sums of the
    others keep their bits, on either side of the 2^12 below the largest
    weight from which on each frame is scaled by itself.  Their errors are those of the same weights
    without it, for which the 2-norm of |B|^2's relative error is about
    1e-7 (two roundings of 2^-24 per value of each of the 9 + 3 stages, added
    in squares: 2 * sqrt(12 / 3) * 2^-24 / sqrt(2) = 1.7e-7 at most)."""
    rng = np.random.default_rng(6)
    v = _volts(2, 1, 64, 12)
    v[:, :, :, 7, 1] = 0
    h = rng.uniform(0.2, 1.3, (256, 4))
    if gains:
        h = h * np.exp(1j * rng.uniform(-np.pi, np.pi, (256, 4)))
    h[7, 1] = strong
    h = h.astype(np.complex64 if gains else np.float32)
    got = _run(v, h, 16, gains=gains)
    ref = orc.beamform_fft(v, 4, 512, 16, taper=h.astype(np.complex128 if gains else np.float64))
    assert np.linalg.norm(got - ref) < 1.7e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("spread", [3.0, 9.0])
def test_wide_range_of_weights(gains, spread):
    """Weights over several decades, with zeros among them and a block whose
    samples are all zero (frames without a largest value)."""
    rng = np.random.default_rng(8)
    v = _volts(2, 2, 48, 13)
    v[16:32, 0] = 0
    h = np.exp(spread * rng.normal(size=(256, 4))) * (rng.random((256, 4)) < 0.8)
    if gains:
        h = h * np.exp(1j * rng.uniform(-np.pi, np.pi, (256, 4)))
    h = h.astype(np.complex64 if gains else np.float32)
    got = _run(v, h, 16, gains=gains)
    ref = orc.beamform_fft(v, 4, 512, 16, taper=h.astype(np.complex128 if gains else np.float64))
    assert not np.any(got[1, 0])
    live = ref > 0
    assert rel_err(got[live], ref[live]) < TOL_FP32
