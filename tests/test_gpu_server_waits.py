"""The server's host calls beside a caller's stream that is busy for long: a
submission that wraps the staging memory, and results copied on many streams,
do not wait for the caller's work; a copy recorded into a graph leaves the
server as it was."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _setup(budget=8 << 20):
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(4)
    v = torch.from_numpy(r.integers(0, 256, (64, 2, 1, 16, 4), dtype=np.uint8)).cuda()
    plan = bf.Plan(n_ns=16, n_chan=2, n_pol=1, block=16)
    srv = bf.Server(plan, ring_samples=64, hbm_budget=budget)
    assert srv.advance(64, v) == bf.BF_OK
    torch.cuda.synchronize()
    return torch, bf, r, v, plan, srv


def _busy(torch, stream, x):
    """About half a second of work on `stream`."""
    with torch.cuda.stream(stream):
        for _ in range(500):
            torch.mm(x, x, out=_busy.out)


def _operand(torch):
    x = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    _busy.out = torch.empty_like(x)
    torch.mm(x, x, out=_busy.out)
    torch.cuda.synchronize()
    return x


def test_staging_memory_wraps_while_a_caller_is_busy():
    torch, bf, r, v, plan, srv = _setup()
    x = _operand(torch)
    ds = [r.uniform(-0.9, 0.9, (4096, 2)) for _ in range(17)]        # 64 KiB of pointings each
    for d in ds[:10]:
        rid = srv.submit(d, 0, 1, 16)
        assert srv.wait(rid)[0] == bf.BF_OK
        if d is not ds[9]:
            assert srv.release(rid) == bf.BF_OK
    side = torch.cuda.Stream()
    dst = torch.empty((1, 1, 1, 4096), device="cuda")
    torch.cuda.synchronize()
    _busy(torch, side, x)
    assert bf.lib().bf_server_copy_result(srv.handle, rid, dst.data_ptr(), side.cuda_stream) == bf.BF_OK
    assert srv.release(rid) == bf.BF_OK
    t0 = time.perf_counter()
    ids = [srv.submit(d, 0, 1, 16) for d in ds[10:]]
    took = time.perf_counter() - t0
    busy = not side.query()
    for d, rid in zip(ds[10:], ids):
        assert srv.wait(rid)[0] == bf.BF_OK
        want = bf.form_tied_beams_v(plan, v[48:].contiguous(), 0, 1, torch.from_numpy(d).cuda())
        assert torch.equal(srv.result(rid), want)
    want = bf.form_tied_beams_v(plan, v[48:].contiguous(), 0, 1, torch.from_numpy(ds[9]).cuda())
    assert torch.equal(dst, want)
    srv.close()
    plan.close()
    print("seven submissions took %.1f ms" % (1e3 * took))
    assert busy and took < 0.1


def test_results_on_many_streams():
    torch, bf, r, v, plan, srv = _setup()
    x = _operand(torch)
    d = r.uniform(-0.9, 0.9, (8, 2))
    rid = srv.submit(d, 0, 2, 64)
    assert srv.wait(rid)[0] == bf.BF_OK
    streams = [torch.cuda.Stream() for _ in range(24)]
    outs = [torch.zeros((4, 2, 1, 8), device="cuda") for _ in streams]
    torch.cuda.synchronize()
    took = 0.0
    for k, (s, o) in enumerate(zip(streams, outs)):
        if k == 20:
            _busy(torch, s, x)
        t0 = time.perf_counter()
        assert bf.lib().bf_server_copy_result(srv.handle, rid, o.data_ptr(), s.cuda_stream) == bf.BF_OK
        took = max(took, time.perf_counter() - t0)
    busy = not streams[20].query()
    assert srv.release(rid) == bf.BF_OK
    # the memory is taken again at once: the copies still hold the first request's beams
    rid = srv.submit(r.uniform(-0.9, 0.9, (8, 2)), 0, 2, 64)
    assert srv.wait(rid)[0] == bf.BF_OK
    torch.cuda.synchronize()
    want = bf.form_tied_beams_v(plan, v, 0, 2, torch.from_numpy(d).cuda())
    assert all(torch.equal(o, want) for o in outs)
    srv.close()
    plan.close()
    print("the longest copy call took %.2f ms" % (1e3 * took))
    assert busy and took < 0.1


def test_more_reads_than_the_server_keeps_events_for():
    """Hundreds of copies behind a busy stream, then the memory given back and
    taken by the next request."""
    torch, bf, r, v, plan, srv = _setup(64 * 1024)
    x = _operand(torch)
    d = r.uniform(-0.9, 0.9, (512, 2))
    rid = srv.submit(d, 0, 2, 64)
    assert srv.wait(rid)[0] == bf.BF_OK
    side = torch.cuda.Stream()
    outs = torch.zeros((200, 4, 2, 1, 512), device="cuda")
    torch.cuda.synchronize()
    _busy(torch, side, x)
    for o in outs:
        assert bf.lib().bf_server_copy_result(srv.handle, rid, o.data_ptr(), side.cuda_stream) == bf.BF_OK
    assert srv.release(rid) == bf.BF_OK
    rid = srv.submit(r.uniform(-0.9, 0.9, (512, 2)), 0, 2, 64)
    assert srv.wait(rid)[0] == bf.BF_OK
    torch.cuda.synchronize()
    want = bf.form_tied_beams_v(plan, v, 0, 2, torch.from_numpy(d).cuda())
    assert torch.equal(outs, want.expand_as(outs))
    srv.close()
    plan.close()
