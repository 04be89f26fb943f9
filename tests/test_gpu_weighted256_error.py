"""Weighted FP32 intensities of the 4 x 256 lattice against 64 bits: the matrix
cores' two FP16 terms per operand leave them no further off than the same
calculation with every operand and sum in FP32.

That calculation, on the CPU: weighted E-W sums and a single-precision 512-point
FFT, the block sum by fused multiply-adds of the real and imaginary parts."""
import numpy as np
import pytest
import scipy.fft

import oracle as orc
import synthgen as sg

pytestmark = pytest.mark.gpu


def _single(v, w, block):
    """[blk][chan][pol][4][512] intensities with FP32 operands and sums."""
    x = (orc.decode_int4(v).astype(np.complex64) * w.astype(np.complex64)).astype(np.complex64)
    a, b = x[..., 0] + x[..., 2], x[..., 0] - x[..., 2]
    c, d = x[..., 1] + x[..., 3], x[..., 1] - x[..., 3]
    d = (-1j * d).astype(np.complex64)
    e = np.stack([a + c, b + d, a - c, b - d], axis=-2)              # [t][chan][pol][4][256]
    z = scipy.fft.fft(e, n=512, axis=-1)
    assert z.dtype == np.complex64
    z = z.reshape((-1, block) + z.shape[1:])
    acc = np.zeros((z.shape[0],) + z.shape[2:], np.float32)
    for t in range(block):
        for part in (z[:, t].imag, z[:, t].real):
            acc = (acc.astype(np.float64) + part.astype(np.float64) ** 2).astype(np.float32)   # one rounding
    return acc * np.float32(1.0 / 1024)


@pytest.mark.parametrize("gains", [False, True])
@pytest.mark.parametrize("block,n_blk", [(4, 16), (16, 8), (80, 2), (160, 1)])
def test_no_further_off_than_single_precision(gains, block, n_blk):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(block)
    v = sg.volts(sg.custom_workload(n_ew=4, n_ns=256, n_chan=4, n_pol=2, n_time=block * n_blk, seed=block, n_src=2,
                                    snr=10.0))
    if gains:
        w = (np.exp(0.1 * r.standard_normal((256, 4))) * np.exp(1j * r.uniform(-np.pi, np.pi, (256, 4)))).astype(np.complex64)
    else:
        g = [np.exp(-0.5 * ((np.arange(n) - (n - 1) / 2) / (0.4 * n)) ** 2) for n in (256, 4)]
        w = np.outer(*g).astype(np.float32)
    plan = bf.Plan(n_ns=256, n_chan=4, n_pol=2, block=block)
    t = torch.from_numpy(w).cuda()
    got = bf.beamform_fft(plan, torch.from_numpy(v).cuda(), **({"gains": t} if gains else {"taper": t})).cpu().numpy()
    plan.close()
    ref = orc.beamform_fft(v, 4, 512, block, taper=w.astype(np.complex128 if gains else np.float64))
    single = _single(v, w, block)
    assert single.shape == ref.shape == got.shape

    def err(x):
        x = x.astype(np.float64) - ref
        return np.linalg.norm(x) / np.linalg.norm(ref), np.sqrt(np.mean((x / ref) ** 2))
    print("2-norm, rms of the relative error: %.3e %.3e, single precision %.3e %.3e" % (err(got) + err(single)))
    assert err(got)[0] <= err(single)[0] and err(got)[1] <= err(single)[1]
