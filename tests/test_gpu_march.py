"""The staged form's marching residual step against the FP64 oracle (every order it serves) and,
bit for bit, against the fused kernel: run ends, ragged tiles, mirrors."""
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

PPP = ("periodic",) * 3
# (nx, ny, nz) that the launch rule gives to the marching kernel; the last run is short in some
SHAPES = [(112, 112, 112), (130, 97, 75), (97, 161, 90), (256, 40, 131)]


def _solver(shape, order, dtype, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    s = sbli.Solver(shape, order=order, dtype=dtype, bc=bc, **synth.TGV)
    q = s.tgv_init(s.empty_state())
    g = torch.Generator(device="cuda").manual_seed(order)
    q.mul_(1 + 0.05 * torch.rand(q.shape, generator=g, device="cuda", dtype=q.dtype))
    return torch, s, q


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", [PPP, ("symmetry",) * 3])
@pytest.mark.parametrize("dtype,order", [("f64", 6), ("f64", 8), ("f32", 6), ("f32", 8)])
def test_march_equals_fused(shape, bc, dtype, order):
    torch, s, q0 = _solver(shape, order, dtype, bc)
    out = []
    for v in (0, len(s.variants()) - 1):
        s.set_tuning(v, shape[2])
        q = q0.clone()
        R = s.rhs(q)
        s.rk3_step(q, s.empty_state(), s.empty_state(), 1e-4, 2)
        out.append((R, q))
    torch.cuda.synchronize()
    s.close()
    assert torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1)])
@pytest.mark.parametrize("order", [8, 10, 12])
def test_march_residual_matches_oracle(oracle_mod, order, bc):
    """The bound of the staged form's other oracle tests, 1e-12 of a field's largest residual."""
    import torch
    import paper_1609_01277_amd as sbli
    from test_gpu_high_order import TOL64, rel_err
    shape = (130, 97, 75)
    q0 = synth.random_conservative_state(shape, seed=40 + order, mom=0.3)
    s = sbli.Solver(shape, order=order, bc=bc, **synth.TGV)
    s.set_tuning(len(s.variants()) - 1, 1)
    R = s.rhs(torch.from_numpy(q0).cuda()).cpu().numpy()
    s.close()
    errs = rel_err(R, oracle.rhs(q0, oracle.Params(n=shape, order=order, bc=bc, **synth.TGV)))
    assert max(errs) <= TOL64, errs
