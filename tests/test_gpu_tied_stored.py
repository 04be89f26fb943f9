"""Tied beams from stored complex FFT beams of the 4 x 32 ... 4 x 256 lattices
(m_ns = 64 ... 512: FP32 operands as three BF16 terms on the matrix cores)
against the definition B_p = sum_{e,A} c_e c_A B[e][A] in FP64.

Tolerance per output, derived: the sums run through at most 6 M / 16 FP32
accumulations of 32 products along N-S and a few roundings of the weights and
of the E-W sum, so |error| <= (6 M / 16 + 48) 2^-24 S with
S = sum |c_e| |c_A| |B|.  An intensity sums |B_p|^2 over T = block * pols samples:
|error| <= sum (2 |B_p| d + d^2) + 2 T 2^-24 sum |B_p|^2 with d the bound on B_p.
"""
import math

import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def _weights(torch, y, m, n):
    A = torch.arange(m, device="cuda", dtype=torch.float64)[None, :, None]
    a = torch.arange(n, device="cuda", dtype=torch.float64)[None, None, :]
    ph = 2 * math.pi * a * (A / m - y[:, None, None])
    return torch.complex(ph.cos().sum(-1) / m, ph.sin().sum(-1) / m)


def _reference(torch, beams, d, dl, n_ns):
    """(B_p, S) of beams [t][chan][pol][4][m]: complex128 and float64 [t][chan][pol][P]."""
    m = 2 * n_ns
    ce, cn = _weights(torch, d[:, 0] * dl, 4, 4), _weights(torch, d[:, 1] * dl, m, n_ns)
    b = beams.to(torch.complex128)
    z = torch.matmul(b.reshape(-1, m), cn.T.contiguous()).reshape(*b.shape[:-1], -1)
    s = torch.matmul(b.abs().reshape(-1, m), cn.abs().T.contiguous()).reshape(*b.shape[:-1], -1)
    return (z * ce.T).sum(-2), (s * ce.abs().T).sum(-2)


def _case(torch, seed, n_time, n_chan, n_pol, n_ns, n_point, scale=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    b = torch.randn((n_time, n_chan, n_pol, 4, 2 * n_ns, 2), generator=g, device="cuda", dtype=torch.float64) * scale
    d = torch.rand((n_point, 2), generator=g, device="cuda", dtype=torch.float64) * 1.6 - 0.8
    d[0] = 0.0
    return torch.view_as_complex(b).to(torch.complex64).contiguous(), d


@pytest.mark.parametrize("n_ns", [32, 64, 128, 256])
@pytest.mark.parametrize("n_point,block,n_blk,pol_sum", [
    (1, 4, 1, False),        # one pointing, one quad: a single live wavefront
    (17, 8, 3, True),        # a second tile with one pointing, units shared by two wavefronts
    (48, 16, 5, False),      # whole tiles, shared by four, a ragged last workgroup
    (65, 20, 2, True),       # five tiles, five quads over four wavefronts
    (70, 16, 260, False),    # as many units as wavefronts in flight: none shared
])
def test_intensities(n_ns, n_point, block, n_blk, pol_sum):
    import torch
    import paper_1710_08591_amd as bf
    beams, d = _case(torch, 7 + n_ns + n_point, block * n_blk, 3, 2, n_ns, n_point)
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=2, n_chan=3, block=block, pol_sum=pol_sum)
    got = bf.form_tied_beams(plan, beams, 1, 2, d).double()
    plan.close()
    ref, s = _reference(torch, beams[:, 1:], d, 0.5, n_ns)
    e = (6 * 2 * n_ns / 16 + 48) * EPS * s
    p = ref.abs() ** 2
    tol = 2 * ref.abs() * e + e * e + 2 * block * (2 if pol_sum else 1) * EPS * p
    p, tol = (v.reshape(n_blk, block, 2, 2, n_point).sum(1) for v in (p, tol))
    if pol_sum:
        p, tol = p.sum(2), tol.sum(2)
    assert got.numel() == p.numel()
    assert bool(((got.reshape(p.shape) - p).abs() <= tol).all())


@pytest.mark.parametrize("n_ns", [32, 256])
@pytest.mark.parametrize("n_time,n_point,scale", [(7, 33, 1.0), (4, 16, 1e-35), (5, 3, 1e37)])
def test_complex_scales(n_ns, n_time, n_point, scale):
    """Complex beams with a ragged last quad; beams near the ends of the FP32 range."""
    import torch
    import paper_1710_08591_amd as bf
    beams, d = _case(torch, n_time, n_time, 2, 2, n_ns, n_point, scale)
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=2, n_chan=2, block=16)
    got = bf.form_tied_beams(plan, beams, 0, 2, d, kind=bf.BF_OUT_COMPLEX).to(torch.complex128)
    plan.close()
    ref, s = _reference(torch, beams, d, 0.5, n_ns)
    assert bool(((got - ref).abs() <= (6 * 2 * n_ns / 16 + 48) * EPS * s + 2.0 ** -126).all())


@pytest.mark.parametrize("n_ns", [32, 128])
def test_values_that_are_not_finite(n_ns):
    """An infinite or NaN beam reaches its own sample and block only; a beam
    that is finite in FP32 but rounds to infinity in BF16 is summed as it is."""
    import torch
    import paper_1710_08591_amd as bf
    beams, d = _case(torch, 5, 64, 1, 1, n_ns, 19)
    d[0] = 0.03                                     # no weight is exactly zero
    clean = beams.clone()
    beams[3, 0, 0, 1, 5] = float("inf")
    beams[21, 0, 0, 2, 9] = float("nan")
    big = clean.clone()
    big[40, 0, 0, 3, 11] = 3.4e38
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=1, n_chan=1, block=16)
    gc = bf.form_tied_beams(plan, beams, 0, 1, d, kind=bf.BF_OUT_COMPLEX)
    gi = bf.form_tied_beams(plan, beams, 0, 1, d)
    gb = bf.form_tied_beams(plan, big, 0, 1, d, kind=bf.BF_OUT_COMPLEX)
    plan.close()
    fin = torch.isfinite(torch.view_as_real(gc)).all(-1).reshape(64, 19)
    assert not bool(fin[3].any()) and not bool(fin[21].any())
    keep = torch.ones(64, dtype=torch.bool, device="cuda")
    keep[3] = keep[21] = False
    assert bool(fin[keep].all())
    gi = torch.isfinite(gi).reshape(4, 19)
    assert not bool(gi[:2].any()) and bool(gi[2:].all())
    ref, s = _reference(torch, clean, d, 0.5, n_ns)
    tol = (6 * 2 * n_ns / 16 + 48) * EPS * s
    assert bool(((gc.to(torch.complex128) - ref).abs() <= tol)[keep].all())
    ref, s = _reference(torch, big, d, 0.5, n_ns)
    assert bool(((gb.to(torch.complex128) - ref).abs() <= (6 * 2 * n_ns / 16 + 48) * EPS * s).all())
