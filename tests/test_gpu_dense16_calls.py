"""FP16 plans of the 4 x 16 lattice: a block's intensities do not depend on how
many blocks the call has, so a stream may be cut into calls anywhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chan,n_pol,block,n_blk", [
    (241, 1, 16, 18), (64, 2, 48, 40), (64, 2, 64, 40), (64, 2, 80, 40), (31, 1, 32, 150), (16, 2, 32, 150)])
def test_calls_of_any_length(n_chan, n_pol, block, n_blk):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(block)
    v = torch.from_numpy(r.integers(0, 256, (block * n_blk, n_chan, n_pol, 16, 4), dtype=np.uint8)).cuda()
    plan = bf.Plan(n_ns=16, n_chan=n_chan, n_pol=n_pol, block=block, precision=bf.BF_PREC_FP16_MFMA)
    whole = bf.beamform_fft(plan, v)
    parts = [bf.beamform_fft(plan, v[a * block:b * block].contiguous()) for a, b in ((0, 1), (1, 4), (4, n_blk))]
    plan.close()
    assert torch.equal(whole, torch.cat(parts))
