"""Dense regridding on the matrix cores (FP32 operands as three BF16 terms) at
the edges of its tiles, against the same contraction in FP64.

Tolerance per output, derived: the weights are FP64 values rounded to FP32
(2^-24 each, and again for the E-W weights), and the sum runs through at most
6 M / 32 FP32 accumulations of 32 products each, so
|error| <= (6 M / 32 + 48) 2^-24 sum |w| |I| (+ the smallest normal number).
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def _weights(torch, y, n, m):
    u = y[:, None] - torch.arange(m, device="cuda", dtype=torch.float64)[None] / m
    d = torch.arange(1, n, device="cuda", dtype=torch.float64)
    return (1 + 2 * torch.cos(2 * math.pi * u[..., None] * d).sum(-1)) / m


def _run(torch, n_ns, m_ew, n_chan, n_blk, n_target, scale=1.0, edit=None):
    import paper_1710_08591_amd as bf
    m, rng = 2 * n_ns, np.random.default_rng(n_ns + n_target + n_blk)
    g = torch.Generator(device="cuda")
    g.manual_seed(n_blk)
    x = (torch.rand((n_blk, n_chan, 1, m_ew, m), generator=g, device="cuda", dtype=torch.float64) ** 4 * scale).float()
    if edit:
        edit(x)
    d = rng.uniform(-0.9, 0.9, (n_target, 2))
    d[0] = 0.0
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=1, n_chan=n_chan, block=16, m_ew=m_ew)
    rg = bf.Regrid2D(plan, d) if m_ew == 8 else bf.Regrid(plan, d[:, 1].copy())
    got = rg(x).double().reshape(n_blk, n_chan, -1, n_target)
    plan.close()
    dd = torch.from_numpy(d).cuda()
    wn = _weights(torch, 0.5 * dd[:, 1], n_ns, m)
    xd = x.double().reshape(-1, m)
    ref = torch.matmul(xd, wn.T.contiguous()).reshape(n_blk, n_chan, m_ew, n_target)
    mag = torch.matmul(xd.abs(), wn.abs().T.contiguous()).reshape(ref.shape)
    if m_ew == 8:
        we = _weights(torch, 0.5 * dd[:, 0], 4, 8).T
        ref, mag = (ref * we).sum(2, keepdim=True), (mag * we.abs()).sum(2, keepdim=True)
    return got, ref, (6 * m / 32 + 48) * EPS * mag + 2.0 ** -126


@pytest.mark.parametrize("n_ns", [16, 32, 64, 256])
@pytest.mark.parametrize("m_ew,n_chan,n_blk,n_target", [
    (4, 1, 1, 1),          # a quarter of a row tile, one target
    (8, 3, 17, 33),        # few rows: one wavefront per tile, 2-D
    (4, 5, 130, 64),       # 64 targets, 64 rows to a workgroup, a ragged last one
    (8, 2, 260, 49),       # 64 targets, a dead tile in the last pair
    (4, 7, 1300, 17),      # 64 targets, 128 rows to a workgroup
    (8, 1, 260, 257),      # a second group of 256 targets that holds one
    (4, 3, 100, 97),       # 256 targets, tiles without targets
    (8, 9, 520, 200),      # 256 targets, sixteen wavefronts
])
def test_tiles(n_ns, m_ew, n_chan, n_blk, n_target):
    import torch
    got, ref, tol = _run(torch, n_ns, m_ew, n_chan, n_blk, n_target)
    assert got.shape == ref.shape
    assert bool(((got - ref).abs() <= tol).all())


@pytest.mark.parametrize("n_blk,n_target", [(3, 20), (600, 40), (300, 150)])
def test_values_beyond_bf16(n_blk, n_target):
    """Intensities near the ends of the FP32 range, infinite and NaN ones: every
    row as the FP32 instructions sum it, other rows untouched."""
    import torch
    got, ref, tol = _run(torch, 64, 4, 2, n_blk, n_target, scale=1e-35)
    assert bool(((got - ref).abs() <= tol).all())

    def edit(x):
        x[0, 0, 0, 0, 3] = 3.4e38
        x[1, 1, 0, 1, 5] = float("inf")
        x[2, 0, 0, 3, 127] = float("nan")
    got, ref, tol = _run(torch, 64, 4, 2, n_blk, n_target, edit=edit)
    bad = ~torch.isfinite(got).all(-1)
    assert bad.nonzero().tolist() == [[1, 1, 1], [2, 0, 3]]
    assert bool(((got - ref).abs() <= tol)[~bad].all())
