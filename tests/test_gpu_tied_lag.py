"""GPU parity of the stacked-visibility tied beams (k_tied_lag.hip) at the edges
of their runs, segments, pointing tiles and integer ranges, against the FP64
oracle's direct phased sums."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu


def _check(n_chan, n_pol, block, n_blk, n_point, pol_sum=False, chan_lo=0, n_sub=None, volts=None, seed=0):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng([seed, n_chan, n_pol, block, n_blk, n_point])
    n_sub = n_chan - chan_lo if n_sub is None else n_sub
    if volts is None:
        volts = r.integers(0, 256, (block * n_blk, n_chan, n_pol, 16, 4), dtype=np.uint8)
    dl = r.uniform(0.3, 0.9, (n_chan, 2))
    d = r.uniform(-1.0, 1.0, (n_point, 2))
    d[0] = 0.0
    plan = bf.Plan(n_ns=16, n_chan=n_chan, n_pol=n_pol, block=block, pol_sum=pol_sum, d_over_lambda=dl)
    got = bf.form_tied_beams_v(plan, torch.from_numpy(volts).cuda(), chan_lo, n_sub,
                               torch.from_numpy(d).cuda()).cpu().numpy().astype(np.float64)
    plan.close()
    chans = np.arange(chan_lo, chan_lo + n_sub)
    ref = orc.tied_intensity(volts[:, chan_lo:chan_lo + n_sub], d, dl, block, chans=chans)
    total = (orc.decode_int4(volts[:, chan_lo:chan_lo + n_sub]).__abs__() ** 2).reshape(n_blk, block, n_sub, n_pol, 64)
    total = total.sum(axis=(1, 4))                       # R_0
    if pol_sum:
        ref, total = ref.sum(axis=2), total.sum(axis=2)
    assert got.shape == ref.shape
    # one rounding to FP32 (2^-24 of the value), and the weights' step: 217
    # weights, each within 2^-30, on |R_d| <= R_0, over n = 64
    tol = 2.0 ** -24 * 1.01 * ref + 217 * 2.0 ** -30 / 64 * total[..., None]
    assert np.all(np.abs(got - ref) <= tol)


@pytest.mark.parametrize("n_chan,n_pol,block,n_blk,n_point,pol_sum", [
    (1, 1, 16, 1, 1, False),
    (3, 2, 16, 33, 17, False),      # one block past a table, one pointing past a wavefront
    (2, 1, 48, 31, 64, False),
    (2, 2, 32, 16, 65, True),       # summed polarisations, a second pointing tile
    (1, 2, 528, 2, 5, True),        # segments: 512 samples' worth over both polarisations
    (1, 1, 1040, 3, 3, False),
])
def test_edges(n_chan, n_pol, block, n_blk, n_point, pol_sum):
    _check(n_chan, n_pol, block, n_blk, n_point, pol_sum)


def test_channel_range_and_long_runs():
    _check(5, 1, 16, 70, 20, chan_lo=2, n_sub=2)
    _check(64, 1, 16, 2100, 70)     # runs of several tables, the last one short


@pytest.mark.parametrize("byte", [0x00, 0x88, 0x77, 0x78, 0x81])
def test_extreme_voltages(byte):
    """Constant voltages, the largest of either sign among them, through the
    longest segment."""
    v = np.full((1024, 1, 2, 16, 4), byte, dtype=np.uint8)
    _check(1, 2, 512, 2, 9, volts=v)
    _check(1, 2, 1024, 1, 9, pol_sum=True, volts=v)


def test_server_ring_wrap_inside_a_group():
    """Windows that start at any sample of the ring, so a 16-sample group may
    straddle its end: equal to the beams straight from the same voltages."""
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(3)
    dl = r.uniform(0.3, 0.9, (4, 2))
    v = torch.from_numpy(r.integers(0, 256, (320, 4, 1, 16, 4), dtype=np.uint8)).cuda()
    d = r.uniform(-1.0, 1.0, (70, 2))
    plan = bf.Plan(n_ns=16, n_chan=4, n_pol=1, block=16, d_over_lambda=dl)
    srv = bf.Server(plan, ring_samples=160, hbm_budget=1 << 24, blocks_per_tile=3)
    at = 0
    for step in (160, 5, 9, 48, 23):
        for k in range(0, step, 80):
            n = min(80, step - k)
            assert srv.advance(n, v[at:at + n].contiguous()) == bf.BF_OK
            at += n
        rid = srv.submit(d, 1, 3, 160 if step != 9 else 96)
        assert srv.wait(rid)[0] == bf.BF_OK
        got = srv.result(rid).cpu().numpy()
        n = got.shape[0] * 16
        want = bf.form_tied_beams_v(plan, v[at - n:at].contiguous(), 1, 3, torch.from_numpy(d).cuda()).cpu().numpy()
        assert np.array_equal(got, want)
        assert srv.release(rid) == bf.BF_OK
    srv.close()
    plan.close()


def test_server_memory_reused_while_a_result_is_read():
    """Results copied on a caller's stream that is still busy, their memory
    given back and taken by the next requests at once: every copy holds its
    own request's beams (the pool fits one request)."""
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(11)
    v = torch.from_numpy(r.integers(0, 256, (512, 8, 1, 16, 4), dtype=np.uint8)).cuda()
    plan = bf.Plan(n_ns=16, n_chan=8, n_pol=1, block=16)
    ds = [r.uniform(-1.0, 1.0, (128, 2)) for _ in range(6)]
    srv = bf.Server(plan, ring_samples=512, hbm_budget=200 * 1024)
    assert srv.advance(512, v) == bf.BF_OK
    side = torch.cuda.Stream()
    x = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    outs = []
    with torch.cuda.stream(side):
        for d in ds:
            rid = srv.submit(d, 0, 8, 512)
            assert srv.wait(rid)[0] == bf.BF_OK
            for _ in range(4):
                x = x @ x * 1e-3               # the copy below waits behind this
            outs.append(srv.result(rid))
            assert srv.release(rid) == bf.BF_OK
    torch.cuda.synchronize()
    for d, o in zip(ds, outs):
        want = bf.form_tied_beams_v(plan, v, 0, 8, torch.from_numpy(d).cuda())
        assert torch.equal(o, want)
    srv.close()
    plan.close()
