"""The launch configuration a context starts with: on every side of its rule (small and large
tiles, one-plane chunks, the staged form) the steps are those of variant 0 bit for bit."""
import pytest

import synth

pytestmark = pytest.mark.gpu

SHAPES = [(17, 18, 19), (33, 32, 40), (50, 47, 65), (96, 96, 96), (97, 98, 99), (130, 120, 70)]
PPP = ("periodic",) * 3
SPS = ("symmetry", "periodic", "symmetry")


def _sbli():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    return sbli, torch


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("order,bc", [(2, PPP), (4, SPS), (6, PPP), (8, SPS)])
def test_default_configuration_is_bitwise_variant_0(shape, dtype, order, bc):
    sbli, torch = _sbli()
    s = sbli.Solver(shape, order=order, dtype=dtype, bc=bc, **synth.TGV)
    v, zc = s.get_tuning()
    assert 0 <= v < len(s.variants()) and 1 <= zc <= shape[2]
    q0 = s.tgv_init(s.empty_state())
    out = []
    for pick in (None, 0):
        if pick is not None:
            s.set_tuning(pick, shape[2])
        q = q0.clone()
        R = s.rhs(q)
        s.rk3_step(q, s.empty_state(), s.empty_state(), 1e-3, 2)
        out.append((R, q))
    torch.cuda.synchronize()
    assert torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    s.close()


@pytest.mark.parametrize("sizes,count,order", [((17,), 1, 8), ((24, 33), 3, 6), ((20, 64, 96), 7, 2), ((40,), 40, 4)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_default_batch_configuration_equals_sequential(sizes, count, order, dtype):
    sbli, torch = _sbli()
    b = sbli.Batch(synth.batch_instances(count=count, seed=3, sizes=sizes), order=order, dtype=dtype)
    q0 = b.tgv_init(b.empty_state())
    ref, got = q0.clone(), q0.clone()
    b.step_sequential(ref, b.empty_state(), b.empty_state(), 2)
    b.step(got, b.empty_state(), b.empty_state(), 2)
    torch.cuda.synchronize()
    assert torch.isfinite(got).all() and torch.equal(got, ref)
