"""Weak tied beams beside a strong coherent source (k_tied_lag.hip): pointings
far down the side lobes of a source without noise, against the FP64 oracle's
direct phased sums (amplitudes, so their own error is far below).

Beams below 2^-14 of R_0 (a coherent source's peak) have their 217 weights to
2^-61 and to the FP64 arithmetic that makes them, a chain of at most 16
roundings of 2^-53 on weights of up to 2: an error of
217 * 2 * 16 * 2^-53 / 64 * R_0 at most, and one rounding to FP32."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu

FLOOR = 217 * 2 * 16 * 2.0 ** -53 / 64
SEEN = 2.0 ** -14


def _volts(kind, n_time, n_pol):
    v = np.full((n_time, 2, n_pol, 16, 4), 0x70, dtype=np.uint8)
    if kind == "turned":                              # the source half a beam off the grid's corner
        sign = np.where((np.arange(16)[:, None] + np.arange(4)) % 2 == 0, 0x70, 0x90).astype(np.uint8)
        v[:] = sign
    elif kind == "weak":                              # the smallest voltages
        v[:] = 0x10
    return v


@pytest.mark.parametrize("kind,block,n_blk,n_pol,pol_sum,server", [
    ("constant", 16, 35, 1, False, False),      # a second table
    ("constant", 16, 35, 1, False, True),
    ("turned", 32, 5, 2, True, False),
    ("weak", 16, 3, 2, False, False),
    ("weak", 16, 3, 2, False, True),
    ("constant", 1040, 2, 1, False, False),     # segments
])
def test_side_lobes(kind, block, n_blk, n_pol, pol_sum, server):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(block + n_pol)
    v = _volts(kind, block * n_blk, n_pol)
    dl = np.full((2, 2), 0.5)
    # nulls of the array are at multiples of 1/8 of sin(theta) along N-S and 1/2 along E-W
    d = np.stack([r.choice([0.0, 0.5, 1.0], 90) - r.choice([0.0, 1.0], 90), r.integers(-8, 9, 90) / 8.0], axis=1)
    d += 10.0 ** r.uniform(-6, -1.5, d.shape) * r.choice([-1.0, 1.0], d.shape)
    plan = bf.Plan(n_ns=16, n_chan=2, n_pol=n_pol, block=block, pol_sum=pol_sum, d_over_lambda=dl)
    if server:
        srv = bf.Server(plan, ring_samples=block * n_blk, hbm_budget=1 << 24, blocks_per_tile=32)
        assert srv.advance(block * n_blk, torch.from_numpy(v).cuda()) == bf.BF_OK
        rid = srv.submit(d, 0, 2, block * n_blk)
        assert srv.wait(rid)[0] == bf.BF_OK
        got = srv.result(rid).cpu().numpy().astype(np.float64)
        srv.close()
    else:
        got = bf.form_tied_beams_v(plan, torch.from_numpy(v).cuda(), 0, 2,
                                   torch.from_numpy(d).cuda()).cpu().numpy().astype(np.float64)
    plan.close()
    ref = orc.tied_intensity(v, d, dl, block, chans=np.arange(2))
    total = (np.abs(orc.decode_int4(v)) ** 2).reshape(n_blk, block, 2, n_pol, 64).sum(axis=(1, 4))[..., None]
    if pol_sum:
        ref, total = ref.sum(axis=2), total.sum(axis=2)
    weak = ref < SEEN * total
    assert weak.mean() > 0.3 and (ref < 1e-9 * total).any()
    err = np.abs(got - ref)
    print("largest error over R_0 of the weak beams: %.2e" % (err / total)[weak].max())
    assert np.all(err[weak] <= (2.0 ** -24 * 1.01 * ref + FLOOR * total)[weak])


def test_no_output_depends_on_its_neighbours():
    """Weak and other outputs side by side, in one call and one by one."""
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(1)
    v = r.integers(0, 256, (16 * 40, 1, 1, 16, 4), dtype=np.uint8)
    v[16 * 7:16 * 20] = 0x70
    v = torch.from_numpy(v).cuda()
    d = np.stack([r.choice([-0.5, 0.0, 0.5], 70), r.integers(-8, 9, 70) / 8.0], axis=1) + 1e-4 * r.standard_normal((70, 2))
    d = torch.from_numpy(d).cuda()
    plan = bf.Plan(n_ns=16, n_chan=1, n_pol=1, block=16)
    whole = bf.form_tied_beams_v(plan, v, 0, 1, d).reshape(40, 70)
    for p in (0, 17, 66):
        for a, b in ((0, 40), (3, 4), (12, 13), (19, 25)):
            part = bf.form_tied_beams_v(plan, v[16 * a:16 * b].contiguous(), 0, 1, d[p:p + 1].contiguous())
            assert torch.equal(part.reshape(-1), whole[a:b, p])
    plan.close()
