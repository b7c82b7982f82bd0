"""The marching residual step where the other tests leave it out: steps at orders 10 and 12 (FP64
keeps part of the z window in LDS there and has one buffer and two barriers a plane), FP32 at those
orders, a closure term, and the split form's plain stores on long rows."""
import numpy as np
import pytest

import oracle
import synth
from oracle import stencil

pytestmark = pytest.mark.gpu

SHAPE = (130, 97, 75)     # ragged tiles, runs of planes of which the last is short
PPP, SSS, SPS = (0, 0, 0), (1, 1, 1), (1, 0, 1)


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    return torch


@pytest.mark.parametrize("bc", [PPP, SSS])
@pytest.mark.parametrize("order", [10, 12])
def test_steps_match_oracle_f64(oracle_mod, order, bc):
    """Two steps; 1e-12 of a field's largest value, the bound of the other oracle tests."""
    torch = _torch()
    import paper_1609_01277_amd as sbli
    from test_gpu_high_order import TOL64, rel_err
    p = oracle.Params(n=SHAPE, order=order, bc=bc, **synth.TGV)
    q0 = synth.random_conservative_state(SHAPE, seed=60 + order, mom=0.3)
    s = sbli.Solver(SHAPE, order=order, bc=bc, **synth.TGV)
    q = s.rk3_step(torch.from_numpy(q0).cuda(), s.empty_state(), s.empty_state(), 1e-4, 2).cpu().numpy()
    s.close()
    errs = rel_err(q, oracle.rk3(q0, p, 1e-4, 2))
    assert max(errs) <= TOL64, errs


def _residual_bound32(q, order):
    """What FP32 may lose of a residual, by field: each neighbour enters products of the size of the
    fluxes with weights a_m / h, c_m / h^2 / Re and a dozen roundings (conversion, nested terms,
    products, sums) of 2^-24."""
    h = [2 * np.pi / n for n in SHAPE]
    w1 = 2 * sum(abs(float(a)) for a in stencil.first_derivative_weights(order))
    w2 = 4 * sum(abs(float(c)) for c in stencil.second_derivative_weights(order)[1])
    s1, s2 = sum(w1 / d for d in h), sum(w2 / d ** 2 for d in h)
    rho, m, E = np.abs(q[0]).max(), np.abs(q[1:4]).max(), np.abs(q[4]).max()
    u, Re, g = m / np.abs(q[0]).min(), synth.TGV["Re"], synth.TGV["gamma"]
    p = (g - 1) * E
    nu = (s2 + s1 ** 2) / Re                       # Laplacian and nested terms
    heat = g / synth.TGV["Pr"] * E / np.abs(q[0]).min() * s2 / Re
    size = [s1 * (m + rho * u)] + [s1 * (m * u + p) + nu * u] * 3 + [s1 * (E + p) * u + nu * u * u + heat]
    return 12 * 2.0 ** -24 * np.array(size)


@pytest.mark.parametrize("bc", [PPP, SPS])
@pytest.mark.parametrize("order", [10, 12])
def test_f32_residual_and_steps(oracle_mod, order, bc):
    torch = _torch()
    import paper_1609_01277_amd as sbli
    p = oracle.Params(n=SHAPE, order=order, bc=bc, **synth.TGV)
    q0 = synth.random_conservative_state(SHAPE, seed=70 + order, mom=0.3).astype(np.float32)
    s = sbli.Solver(SHAPE, order=order, dtype="f32", bc=bc, **synth.TGV)
    qd = torch.from_numpy(q0).cuda()
    R = s.rhs(qd).cpu().numpy().astype(np.float64)
    dt, steps = 1e-4, 2
    q = s.rk3_step(qd, s.empty_state(), s.empty_state(), dt, steps).cpu().numpy().astype(np.float64)
    s.close()
    bound = _residual_bound32(q0.astype(np.float64), order)
    err = np.abs(R - oracle.rhs(q0.astype(np.float64), p)).max(axis=(1, 2, 3))
    print("residual error over its bound:", np.round(err / bound, 3), flush=True)
    assert (err <= bound).all(), err / bound
    # each of six stages rounds the state once and adds dt times a residual's error
    qref = oracle.rk3(q0.astype(np.float64), p, dt, steps)
    qb = 3 * steps * (2.0 ** -23 * np.abs(qref).max(axis=(1, 2, 3)) + dt * bound)
    qerr = np.abs(q - qref).max(axis=(1, 2, 3))
    print("state error over its bound:", np.round(qerr / qb, 3), flush=True)
    assert (qerr <= qb).all(), qerr / qb


@pytest.mark.parametrize("order", [6, 8])
def test_march_adds_the_closure_term(order):
    """128^3, where the staged form marches: bitwise the fused form with the same network."""
    torch = _torch()
    import paper_1609_01277_amd as sbli
    from oracle import nn
    from paper_1609_01277_amd import closure
    n = 128
    net = closure.ClosureNet(n, 1)
    net.set_params(closure.join_params(nn.init_params(np.random.default_rng(4))).astype(np.float32) * 0.05)
    stats = np.zeros(35, dtype=np.float32)
    stats[5:10] = stats[15:20] = 1.0
    stats[20:25] = 1e3
    net.set_stats(stats)
    s = sbli.Solver(n, order=order, dtype="f32", **synth.TGV)
    plain = s.rk3_step(s.tgv_init(s.empty_state()), s.empty_state(), s.empty_state(), 1e-3, 1)
    closure.attach(s, net)
    out = []
    for v in (0, len(s.variants()) - 1):
        s.set_tuning(v, n)
        out.append(s.rk3_step(s.tgv_init(s.empty_state()), s.empty_state(), s.empty_state(), 1e-3, 1))
    assert closure.counts(s) == (6, 0)
    assert torch.equal(out[0], out[1]) and not torch.equal(out[0], plain)
    s.close()
    net.close()


def test_split_form_on_rows_beyond_the_descriptor():
    """16 rows of FP64 values span more than 2^30 bytes: the split form takes plain stores (as the
    marching step does by the same rule) and agrees bitwise with the tiled staged form."""
    torch = _torch()
    import paper_1609_01277_amd as sbli
    n = (2 ** 23 + 24, 9, 9)
    s = sbli.Solver(n, order=4, length=(6.2e5, 6.28, 6.28), **synth.TGV)
    vs = s.variants()
    split = [v for v in range(len(vs) - 1) if vs[v][5] == 2 and vs[v][1] == 16][0]
    g = torch.Generator(device="cuda").manual_seed(9)
    q0 = torch.empty(s.shape, dtype=torch.float64, device="cuda").uniform_(-0.3, 0.3, generator=g)
    q0[0].mul_(0.1).add_(1.0)
    q0[4].add_(179.0)
    out = []
    for v in (split, len(vs) - 1):
        s.set_tuning(v, 9)
        q, qt, dq = q0.clone(), s.empty_state(), s.empty_state()
        s.rk3_step(q, qt, dq, 1e-4, 1)
        del qt, dq
        out.append(q)
        torch.cuda.synchronize()
        print("variant %d %s done" % (v, vs[v]), flush=True)
    assert torch.equal(out[0], out[1]) and not torch.equal(out[0], q0)
    del out, q, q0
    s.close()
    torch.cuda.empty_cache()
