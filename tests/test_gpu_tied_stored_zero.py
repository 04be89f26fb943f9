"""Stored beams that are exactly zero (dead channels, zero-filled gaps): their
complex tied beams are exactly zero and cost no second pass (k_tied_stored.hip),
while beams so small that their BF16 terms vanish are still formed in FP32."""
import pytest

pytestmark = pytest.mark.gpu


def _time(torch, fn):
    for _ in range(3):
        fn()
    best = 1e9
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 3)
    return best


@pytest.mark.parametrize("n_ns,n_point", [(32, 64), (64, 48), (256, 16)])
def test_zero_beams(n_ns, n_point):
    import torch
    import paper_1710_08591_amd as bf
    g = torch.Generator(device="cuda").manual_seed(n_ns)
    n_chan, n_time = 16, 262144 // (16 * n_ns)
    b = torch.view_as_complex(torch.randn((n_time, n_chan, 2, 4, 2 * n_ns, 2), generator=g, device="cuda"))
    d = torch.rand((n_point, 2), generator=g, device="cuda", dtype=torch.float64) * 1.6 - 0.8
    plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=2, n_chan=n_chan, block=16)

    def run(x):
        return bf.form_tied_beams(plan, x, 0, n_chan, d, kind=bf.BF_OUT_COMPLEX)
    gap = b.clone()
    gap[5:22, 3:] = 0
    gap[:, 1, 1] = 0
    live, got = run(b), run(gap)
    shape = (n_time, n_chan, 2, n_point)
    live, got = live.reshape(shape), got.reshape(shape)
    assert not bool(torch.view_as_real(got[5:22, 3:]).any()) and not bool(torch.view_as_real(got[:, 1, 1]).any())
    assert torch.equal(got[22:, 3:], live[22:, 3:]) and torch.equal(got[:, 0], live[:, 0])
    tiny = b * 2.0 ** -140                       # below BF16's range: FP32 holds nine bits or more
    small = run(tiny).reshape(shape)
    ref = live * 2.0 ** -140
    assert bool((small - ref).abs().max() <= 2 * n_ns * 4 * 2.0 ** -148)
    assert bool(torch.view_as_real(small).any())
    zero = torch.zeros_like(b)
    t_live, t_zero = _time(torch, lambda: run(b)), _time(torch, lambda: run(zero))
    plan.close()
    print("live %.1f us, zero %.1f us" % (1e3 * t_live, 1e3 * t_zero))
    assert t_zero < 1.3 * t_live
