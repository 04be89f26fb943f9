"""Tasks without signal among live ones (k_lag.hip takes two tasks through one
complex transform): zeros stay exactly zero, and the weakest possible signal is
not changed by a neighbour at full scale."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(v, n_ns, block, precision=0):
    import torch
    import paper_1710_08591_amd as bf
    plan = bf.Plan(n_ns=n_ns, n_chan=v.shape[1], n_pol=v.shape[2], block=block, precision=precision)
    out = bf.beamform_fft(plan, torch.from_numpy(v).cuda()).cpu().numpy()
    plan.close()
    return out


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("n_ns,n_chan,n_blk", [(16, 300, 15), (64, 50, 24), (256, 40, 8)])
def test_zeros_stay_zero(n_ns, n_chan, n_blk, precision):
    """More tasks than workgroups' rounds hold one of; one polarisation of some
    channels and one whole block without data."""
    r = np.random.default_rng(n_ns)
    block = 16
    v = r.integers(0, 256, (n_blk * block, n_chan, 2, n_ns, 4), dtype=np.uint8)
    v[:, ::3, 1] = 0
    v[:, 1::3, 0] = 0
    v[3 * block:4 * block] = 0
    out = _run(v, n_ns, block, precision)
    assert not out[:, ::3, 1].any() and not out[:, 1::3, 0].any() and not out[3].any()
    assert out[0, 2].any()


@pytest.mark.parametrize("n_ns,n_chan,n_blk", [(16, 300, 15), (256, 40, 8)])
def test_weak_task_beside_a_strong_one(n_ns, n_chan, n_blk):
    """One antenna at 1 in one sample: |B|^2 is 1 in every beam, so the outputs
    are 1 / (4 n) exactly, whatever the other polarisation holds."""
    block = 64
    v = np.full((n_blk * block, n_chan, 2, n_ns, 4), 0x88, dtype=np.uint8)
    v[:, :, 1] = 0
    v[::block, :, 1, 3, 0] = 0x10
    out = _run(v, n_ns, block)
    assert np.all(out[:, :, 1] == np.float32(1.0 / (4 * n_ns)))
    alone = _run(np.ascontiguousarray(v[:block, :1]), n_ns, block)
    assert np.array_equal(out[:1, :1], alone)
