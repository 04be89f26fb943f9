"""The starting beam of the localisation: the lowest index of a row's largest
value, NaN ignored, over ties within a lane's beams, across lanes and rows of
lanes.  With no iteration and a window of one beam the estimate is the beam
itself, sin(theta) = (A/M, wrapped to [-1/2, 1/2)) / (d/lambda), and the peak is
(2 n - 1)/M of its intensity, both to rounding (FP64 estimate, FP32 peak)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ns", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("shift", [0, 1])              # 1: rows that are not 16-byte aligned
def test_lowest_index_of_the_largest(n_ns, shift):
    import torch
    import paper_1710_08591_amd as bf
    m, n_blk = 2 * n_ns, 19                            # 4 x 19 rows: a ragged second wavefront
    rng = np.random.default_rng(n_ns)
    x = rng.uniform(0.0, 1.0, (n_blk * 4, m)).astype(np.float32)
    for r in range(len(x)):
        a = int(rng.integers(m))
        if r % 8 == 1:
            x[r, [a, (a + 1) % m]] = 2.0               # neighbours
        elif r % 8 == 2:
            x[r, [a, (a + m // 2) % m]] = 2.0          # another half of the lanes
        elif r % 8 == 3:
            x[r, [0, m - 1]] = 2.0
        elif r % 8 == 4:
            x[r, a] = np.nan
        elif r % 8 == 5:
            x[r] = -np.inf
        elif r % 8 == 6:
            x[r] = -x[r]
        elif r % 8 == 7:
            x[r] = 0.25
    x[10] = np.nan
    ref = np.zeros(len(x), dtype=int)
    for r in range(len(x)):
        v = np.where(np.isnan(x[r]), -np.inf, x[r])
        ref[r] = int(np.argmax(v))
    buf = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")
    t = buf[shift:shift + x.size].view(n_blk, 1, 1, 4, m)
    t.copy_(torch.from_numpy(x).view(n_blk, 1, 1, 4, m))
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=1, n_chan=1, block=16)
    st, pk = bf.localize(plan, t, n_window=1, n_iter=0)
    plan.close()
    y = ref / m
    want = (np.floor(y + 0.5) * -1.0 + y) / 0.5
    assert np.max(np.abs(st.cpu().numpy().reshape(-1) - want)) < 1e-15
    val = x[np.arange(len(x)), ref]
    ok = np.isfinite(val)
    assert np.allclose(pk.cpu().numpy().reshape(-1)[ok], val[ok] * (2 * n_ns - 1) / m, rtol=2e-7, atol=0)
