"""The staged form's nested-field step in runs of every length its launch rule gives: the
residual is the fused kernel's bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (nx, ny, nz): runs of 1 plane, of 2 with a last run of 1, of a third of the grid and more,
# several tiles with ragged ends
SHAPES = [(17, 17, 17), (40, 33, 70), (130, 40, 31), (96, 97, 51), (33, 260, 33), (161, 170, 37)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,order", [("f64", 8), ("f64", 6), ("f32", 8), ("f32", 4)])
def test_staged_rhs_equals_fused(shape, dtype, order):
    import torch
    import paper_1609_01277_amd as sbli
    import synth
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    s = sbli.Solver(shape, order=order, dtype=dtype, **synth.TGV)
    q, got, ref = s.empty_state(), s.empty_state(), s.empty_state()
    s.tgv_init(q)
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    q.mul_(1 + 0.05 * torch.rand(q.shape, generator=g, device="cuda", dtype=q.dtype))
    s.set_tuning(0, shape[2])
    s.rhs(q, ref)
    s.set_tuning(len(s.variants()) - 1, 1)
    s.rhs(q, got)
    torch.cuda.synchronize()
    s.close()
    assert torch.isfinite(ref).all()
    np.testing.assert_array_equal(got.cpu().numpy(), ref.cpu().numpy())
