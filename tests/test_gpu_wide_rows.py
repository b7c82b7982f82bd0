"""Rows so long that a tile's span passes the stores' buffer descriptor (2^30 bytes): the fused
variants take plain stores there and agree bitwise with the staged form, which has none."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_fused_stores_on_rows_beyond_the_descriptor():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    n = (2 ** 24 + 40, 5, 5)      # 16 rows of FP32 values span more than 2^30 bytes
    s = sbli.Solver(n, order=2, dtype="f32", length=(6.2e5, 6.28, 6.28), **synth.TGV)
    vs = s.variants()
    g = torch.Generator(device="cuda").manual_seed(5)
    q0 = torch.empty(s.shape, dtype=torch.float32, device="cuda")
    q0.uniform_(-0.3, 0.3, generator=g)
    q0[0].mul_(0.1).add_(1.0)
    q0[4].add_(179.0)
    out = []
    tall = [v for v in range(len(vs) - 1) if vs[v][1] == 16]
    for v in (tall[0], tall[-1], len(vs) - 1):
        s.set_tuning(v, 5)
        q, qt, dq = q0.clone(), s.empty_state(), s.empty_state()
        s.rk3_step(q, qt, dq, 1e-4, 1)
        del qt, dq
        R = s.rhs(q0)
        out.append((q, R))
        print("variant %d %s done" % (v, vs[v]), flush=True)
    for q, R in out[:-1]:
        assert torch.equal(R, out[-1][1])
        assert torch.equal(q, out[-1][0])
    assert not torch.equal(out[0][0], q0)
    del out, q, R, q0
    s.close()
    torch.cuda.empty_cache()
