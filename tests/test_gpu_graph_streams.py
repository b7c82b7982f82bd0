"""Graphs captured from one untuned context of order 6 or 8, on buffers of their own, replayed
beside each other on two streams: each replay gives the eager result.  (The staged form, which
sbli_init selects there, keeps its nested fields in the context.)"""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,order,n", [("f64", 6, 48), ("f64", 8, 64), ("f32", 6, 64), ("f32", 8, 48)])
def test_two_graphs_of_one_context(dtype, order, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    streams = [torch.cuda.Stream() for _ in range(2)]
    own = torch.cuda.Stream()
    s = sbli.Solver(n, order=order, dtype=dtype, stream=own, **synth.TGV)
    assert s.get_tuning()[0] == len(s.variants()) - 1          # the staged form by default
    gen = torch.Generator(device="cuda").manual_seed(order)
    with torch.cuda.stream(own):
        q0 = s.tgv_init(s.empty_state())
        starts = [q0 * (1 + 0.02 * torch.rand(q0.shape, generator=gen, device="cuda", dtype=q0.dtype)) for _ in range(2)]
        want = []
        for q in starts:
            e = q.clone()
            want.append((s.rhs(q), s.rk3_step(e, s.empty_state(), s.empty_state(), 1e-3, 3)))
    torch.cuda.synchronize()
    graphs, bufs = [], []
    for q in starts:
        b = dict(q=q.clone(), qt=s.empty_state(), dq=s.empty_state(), R=s.empty_state())
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=own):
            s.rhs(b["q"], b["R"])
            s.rk3_step(b["q"], b["qt"], b["dq"], 1e-3, 3)
        graphs.append(g)
        bufs.append(b)
    for rep in range(5):
        for b, q in zip(bufs, starts):
            b["q"].copy_(q)
        torch.cuda.synchronize()
        for g, st in zip(graphs, streams):
            with torch.cuda.stream(st):
                g.replay()
        with torch.cuda.stream(own):                           # and the context's own eager work beside them
            eager = s.rhs(starts[rep % 2])
        torch.cuda.synchronize()
        assert torch.equal(eager, want[rep % 2][0])
        for b, (R, q) in zip(bufs, want):
            assert torch.equal(b["R"], R) and torch.equal(b["q"], q), (dtype, order, rep)
    s.close()
