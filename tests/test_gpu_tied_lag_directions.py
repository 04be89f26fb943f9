"""Directions that are not finite (k_tied_lag.hip): their beams are NaN, straight
from voltages and through the server, and the other pointings are untouched."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BAD = [(np.nan, 0.1), (0.1, np.nan), (np.inf, 0.0), (0.0, -np.inf), (np.nan, np.nan), (np.inf, -np.inf)]


def _case(n_point, block, n_pol):
    import torch
    r = np.random.default_rng(n_point)
    v = torch.from_numpy(r.integers(0, 256, (block * 35, 3, n_pol, 16, 4), dtype=np.uint8)).cuda()
    d = r.uniform(-0.9, 0.9, (n_point, 2))
    bad = d.copy()
    at = r.permutation(n_point)[:len(BAD)]
    for k, i in enumerate(at):
        bad[i] = BAD[k]
    ok = np.ones(n_point, dtype=bool)
    ok[at] = False
    return torch, v, d, bad, ok


@pytest.mark.parametrize("n_point,block,n_pol,pol_sum", [(6, 16, 1, False), (70, 16, 2, False), (9, 528, 2, True)])
def test_from_voltages(n_point, block, n_pol, pol_sum):
    import paper_1710_08591_amd as bf
    torch, v, d, bad, ok = _case(n_point, block, n_pol)
    plan = bf.Plan(n_ns=16, n_chan=3, n_pol=n_pol, block=block, pol_sum=pol_sum)
    want, got = (bf.form_tied_beams_v(plan, v, 0, 3, torch.from_numpy(x).cuda()).cpu().numpy() for x in (d, bad))
    plan.close()
    assert np.all(np.isnan(got[..., ~ok]))
    assert np.array_equal(got[..., ok], want[..., ok])


def test_through_the_server():
    import paper_1710_08591_amd as bf
    torch, v, d, bad, ok = _case(70, 16, 1)
    plan = bf.Plan(n_ns=16, n_chan=3, n_pol=1, block=16)
    srv = bf.Server(plan, ring_samples=560, hbm_budget=1 << 24, blocks_per_tile=3)
    plan.close()
    assert srv.advance(560, v) == bf.BF_OK
    outs = []
    for x in (d, bad):
        rid = srv.submit(x, 0, 3, 560)
        assert srv.wait(rid)[0] == bf.BF_OK
        outs.append(srv.result(rid).cpu().numpy())
        assert srv.release(rid) == bf.BF_OK
    srv.close()
    assert np.all(np.isnan(outs[1][..., ~ok]))
    assert np.array_equal(outs[1][..., ok], outs[0][..., ok])
