"""GPU parity of the stacked-visibility intensities (k_lag.hip) at the edges of
their tasks, rounds, steps and integer ranges, against the FP64 oracle."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu

# The R_d are exact integers and their transform runs in FP64, so an output is
# the oracle's value rounded once to FP32 (2^-24 of it), up to the FP64
# rounding of a 512-point transform of the two tasks it runs together (well
# under 1e-12 of the largest power among them).
ROUND = 2.0 ** -24 * 1.01
FLOOR = 1e-12


def _check(n_ns, n_chan, n_pol, block, n_blk, pol_sum=False, keep=0, volts=None, precision=0, seed=0):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng([seed, n_ns, n_chan, n_pol, block, n_blk])
    if volts is None:
        volts = r.integers(0, 256, (block * n_blk, n_chan, n_pol, n_ns, 4), dtype=np.uint8)
    sel = r.integers(0, 2 * n_ns, (n_chan, keep)).astype(np.int32) if keep else None
    plan = bf.Plan(n_ns=n_ns, n_chan=n_chan, n_pol=n_pol, block=block, pol_sum=pol_sum, ns_select=sel,
                   precision=precision)
    out = torch.full(plan.out_shape(block * n_blk), -1.0, device="cuda")
    bf.beamform_fft(plan, torch.from_numpy(volts).cuda(), out=out)
    got = out.cpu().numpy().astype(np.float64)
    plan.close()
    ref = orc.beamform_fft(volts, 4, 2 * n_ns, block, ns_select=sel, pol_sum=pol_sum)
    assert got.shape == ref.shape
    assert np.all(np.abs(got - ref) <= ROUND * ref + FLOOR * ref.max())


@pytest.mark.parametrize("n_ns", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("n_chan,n_pol,block,n_blk,pol_sum,keep", [
    (1, 1, 16, 1, False, 0),       # one task
    (3, 1, 4, 5, False, 7),        # a quarter of a step, odd counts, a clamp
    (5, 2, 20, 3, True, 0),        # a ragged second step, summed polarisations
    (3, 2, 48, 2, False, 31),      # three whole steps
    (1, 2, 12, 1, True, 1),
])
def test_edges(n_ns, n_chan, n_pol, block, n_blk, pol_sum, keep):
    _check(n_ns, n_chan, n_pol, block, n_blk, pol_sum, keep)


@pytest.mark.parametrize("n_ns,n_chan,n_blk", [(16, 67, 37), (32, 41, 29), (64, 31, 51), (128, 23, 79), (256, 13, 97)])
def test_many_tasks(n_ns, n_chan, n_blk):
    """More tasks than one per workgroup: two rounds, several per round, and a
    last unit that is not full."""
    _check(n_ns, n_chan, 1, 4, n_blk, keep=9)
    _check(n_ns, n_chan, 2, 16, max(1, n_blk // 4))


@pytest.mark.parametrize("n_ns", [16, 64, 256])
@pytest.mark.parametrize("byte", [0x00, 0x88, 0x77, 0x78, 0x87, 0xF1])
def test_extreme_voltages(n_ns, byte):
    """Constant voltages, the largest of either sign among them (E-W sums of -32)."""
    v = np.full((32, 2, 1, n_ns, 4), byte, dtype=np.uint8)
    _check(n_ns, 2, 1, 16, 2, volts=v)
    v[:, :, :, :, 1::2] = np.uint8((byte & 0x0F) << 4 | byte >> 4)
    _check(n_ns, 2, 1, 32, 1, volts=v)


@pytest.mark.parametrize("n_ns,block", [(16, 32768), (16, 33000), (128, 4096 + 4), (256, 2048), (256, 4112)])
def test_long_blocks(n_ns, block):
    """At and past the sample count where int32 sums are carried on in FP64,
    with the largest voltages."""
    r = np.random.default_rng(block)
    v = np.where(r.random((block, 1, 1, n_ns, 4)) < 0.9, 0x88, 0x77).astype(np.uint8)
    _check(n_ns, 1, 1, block, 1, volts=v)


@pytest.mark.parametrize("precision", [1, 2])
def test_mixed_precision_plans(precision):
    """Unwindowed intensities of the FP16 and FP8 plans take the same exact route."""
    _check(16, 3, 2, 16, 3, keep=5, precision=precision)
    _check(64, 2, 1, 32, 2, precision=precision)
    _check(256, 2, 2, 16, 1, pol_sum=True, precision=precision)
