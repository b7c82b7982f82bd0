"""Variant indices are stored by callers of sbli_set_tuning: each keeps its configuration, stays
accepted and steps to the default's bits."""
import pytest

import synth

pytestmark = pytest.mark.gpu

KEPT = {
    ("f64", 2): [(16, 16, 1, 0, 1, 0, 0), (16, 16, 1, 1, 1, 0, 0), (32, 8, 1, 1, 1, 0, 0), (16, 8, 1, 1, 2, 0, 0),
                 (16, 16, 1, 1, 1, 1, 0)],
    ("f64", 4): [(16, 16, 1, 0, 1, 0, 0), (16, 16, 1, 1, 1, 0, 0), (16, 16, 0, 1, 1, 0, 0), (32, 8, 0, 0, 1, 0, 0),
                 (16, 8, 1, 1, 2, 0, 0), (16, 16, 1, 1, 1, 1, 0), (16, 16, 1, 0, 1, 1, 0)],
    ("f32", 4): [(16, 8, 1, 0, 1, 0, 0), (16, 8, 1, 1, 1, 0, 0), (16, 16, 1, 1, 1, 0, 0), (32, 8, 1, 1, 1, 0, 0),
                 (32, 8, 1, 1, 3, 0, 0), (16, 16, 1, 1, 3, 0, 0), (16, 16, 1, 1, 1, 1, 0), (32, 8, 1, 1, 1, 1, 0),
                 (16, 16, 1, 1, 3, 1, 0), (32, 16, 1, 1, 1, 0, 0), (32, 16, 1, 1, 1, 1, 0)],
}


@pytest.mark.parametrize("dtype,order", sorted(KEPT))
def test_indices_keep_their_configuration(dtype, order):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    n = (37, 26, 33)
    s = sbli.Solver(n, order=order, dtype=dtype, **synth.TGV)
    q0 = s.tgv_init(s.empty_state())
    want = s.rk3_step(q0.clone(), s.empty_state(), s.empty_state(), 1e-3, 1)
    assert [tuple(v) for v in s.variants()[:len(KEPT[dtype, order])]] == KEPT[dtype, order]
    for v in range(len(KEPT[dtype, order])):
        s.set_tuning(v, n[2])
        got = s.rk3_step(q0.clone(), s.empty_state(), s.empty_state(), 1e-3, 1)
        assert torch.equal(got, want), v
    s.close()
