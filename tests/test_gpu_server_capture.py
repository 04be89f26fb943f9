"""A result copy recorded into a graph: the copy runs on each replay, and the
server's own streams stay out of the capture."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_copy_in_a_graph():
    import torch
    import paper_1710_08591_amd as bf
    r = np.random.default_rng(4)
    v = torch.from_numpy(r.integers(0, 256, (64, 2, 1, 16, 4), dtype=np.uint8)).cuda()
    d = r.uniform(-0.9, 0.9, (8, 2))
    plan = bf.Plan(n_ns=16, n_chan=2, n_pol=1, block=16)
    srv = bf.Server(plan, ring_samples=64, hbm_budget=1 << 20)
    assert srv.advance(64, v) == bf.BF_OK
    rid = srv.submit(d, 0, 2, 64)
    assert srv.wait(rid)[0] == bf.BF_OK
    want = bf.form_tied_beams_v(plan, v, 0, 2, torch.from_numpy(d).cuda())
    dst = torch.empty_like(want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        st = bf.lib().bf_server_copy_result(srv.handle, rid, dst.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == bf.BF_OK
    for _ in range(3):
        dst.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dst, want)
    # the server goes on as before
    other = srv.submit(d[:3], 0, 1, 32)
    assert srv.wait(other)[0] == bf.BF_OK
    assert srv.result(other).shape == (2, 1, 1, 3)
    assert srv.release(other) == bf.BF_OK and srv.release(rid) == bf.BF_OK
    again = srv.submit(d, 0, 2, 64)
    assert srv.wait(again)[0] == bf.BF_OK
    assert torch.equal(srv.result(again), want)
    srv.close()
    plan.close()
