"""Localisation with windows of 17 to 64 beams (k_localize.hip passes their rows
through LDS one at a time; that two such workgroups fit a CU is asserted where
the kernel is compiled), against the FP64 oracle on the same FP32 intensities
as in tests/test_gpu_localize.py: 1e-9 in sin(theta), 1e-6 of the peak."""
import numpy as np
import pytest

import oracle as orc
import synthgen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ns,n_window", [
    (16, 17), (16, 31), (32, 64), (64, 17), (64, 63), (128, 33), (128, 64), (256, 17), (256, 48)])
@pytest.mark.parametrize("shift", [0, 1])              # 1: rows that are not 16-byte aligned
def test_wide_windows(n_ns, n_window, shift):
    import torch
    import paper_1710_08591_amd as bf
    n_blk = 3 if n_ns >= 128 else 7
    w = sg.custom_workload(n_ew=4, n_ns=n_ns, n_chan=3, n_pol=2, n_time=16 * n_blk, seed=n_ns + n_window, n_src=3,
                           snr=20.0, dl=(0.4, 0.8))
    x = orc.beamform_fft(sg.volts(w), 4, 2 * n_ns, 16).astype(np.float32)
    buf = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")
    t = buf[shift:shift + x.size].view(x.shape)
    t.copy_(torch.from_numpy(x))
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_chan=3, n_pol=2, block=16, d_over_lambda=w.d_over_lambda())
    st, pk = bf.localize(plan, t, n_window=n_window, n_iter=5)
    plan.close()
    ref_st, ref_pk = orc.localize(x.astype(np.float64), n_ns, w.d_over_lambda()[:, 1], n_window, 5)
    assert np.max(np.abs(st.cpu().numpy() - ref_st)) < 1e-9
    assert np.max(np.abs(pk.cpu().numpy() - ref_pk) / np.abs(ref_pk)) < 1e-6
