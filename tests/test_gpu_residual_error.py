"""Rounding error of the residual, field by field: no larger than that of the plain formulation
(separate derivative sums of Q, Q u, u, p, the nested terms; no fused multiply-add) carried out in
the same type on the CPU.  Both are compared with 80-bit arithmetic on the same inputs.  The bound
follows from counting roundings: D_j(rho u_j) takes the momentum as stored, the velocities are
rounded quotients and 2p is rounded once, each at most what the plain formulation does, and fused
multiply-adds only take roundings away.  The states carry random low bits, so no product is exact
by chance."""
import math

import numpy as np
import pytest

import synth
from oracle import stencil

pytestmark = pytest.mark.gpu

SHAPE = (40, 36, 33)


def _state(seed):
    nx, ny, nz = SHAPE
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*(2 * math.pi * np.arange(n) / n for n in (nz, ny, nx)), indexing="ij")
    ph = rng.uniform(0, 2 * math.pi, 12)
    g, M = synth.TGV["gamma"], synth.TGV["Mach"]
    u = np.sin(x) * np.cos(y) * np.cos(z) + 0.05 * np.sin(2 * x + ph[0]) * np.cos(y + ph[1]) * np.sin(3 * z + ph[2])
    v = -np.cos(x) * np.sin(y) * np.cos(z) + 0.05 * np.cos(x + ph[3]) * np.sin(2 * y + ph[4]) * np.cos(z + ph[5])
    w = 0.05 * np.sin(x + ph[6]) * np.cos(2 * y + ph[7]) * np.sin(z + ph[8])
    rho = 1 + 0.05 * M * np.sin(x + ph[9]) * np.sin(y + ph[10]) * np.cos(2 * z + ph[11])
    p = 1 / (g * M * M) + (np.cos(2 * x) + np.cos(2 * y)) * (np.cos(2 * z) + 2) / 16
    q = np.stack([rho, rho * u, rho * v, rho * w, p / (g - 1) + 0.5 * rho * (u * u + v * v + w * w)])
    return q * (1 + 1e-5 * rng.uniform(-1, 1, q.shape))


def _plain(q, order, ft):
    """The residual by separate sums with every operation rounded to ft; q as stored."""
    r = order // 2
    a = [ft(f.numerator) / ft(f.denominator) for f in stencil.first_derivative_weights(order)]
    c0, c = stencil.second_derivative_weights(order)
    c0, c = ft(c0.numerator) / ft(c0.denominator), [ft(f.numerator) / ft(f.denominator) for f in c]
    prm = synth.TGV
    Re, M, Pr, g = (ft(prm[k]) for k in ("Re", "Mach", "Pr", "gamma"))
    h = [ft(2 * math.pi) / ft(n) for n in SHAPE]
    q = q.astype(ft)
    rho, m, E = q[0], [q[1], q[2], q[3]], q[4]
    one, half, two = ft(1), ft(0.5), ft(2)

    def D(f, d):
        s = np.zeros_like(f)
        for k in range(r, 0, -1):
            s = s + (a[k - 1] / h[d]) * (np.roll(f, -k, 2 - d) - np.roll(f, k, 2 - d))
        return s

    def D2(f, d):
        s = (c0 / (h[d] * h[d])) * f
        for k in range(1, r + 1):
            s = s + (c[k - 1] / (h[d] * h[d])) * (np.roll(f, -k, 2 - d) + np.roll(f, k, 2 - d))
        return s

    rr = one / rho
    u = [mi * rr for mi in m]
    p = (g - one) * (E - half * (m[0] * u[0] + m[1] * u[1] + m[2] * u[2]))
    Tm = g * M * M * p * rr
    G = [[D(u[i], d) for d in range(3)] for i in range(3)]
    th = G[0][0] + G[1][1] + G[2][2]
    V = []
    for d in range(3):
        tau = [(G[i][d] + G[d][i]) / Re - (two / (ft(3) * Re) * th if i == d else ft(0)) for i in range(3)]
        V.append(u[0] * tau[0] + u[1] * tau[1] + u[2] * tau[2])
    R = [np.zeros_like(rho) for _ in range(5)]
    kappa = one / ((g - one) * M * M * Pr * Re)
    for d in range(3):
        dU = D(u[d], d)
        R[0] = R[0] - half * (D(m[d], d) + u[d] * D(rho, d) + rho * dU)
        for i in range(3):
            F = m[i] * u[d] + (two * p if i == d else ft(0))
            R[1 + i] = R[1 + i] - half * (D(F, d) + u[d] * D(m[i], d) + m[i] * dU) + D2(u[i], d) / Re
        R[1 + d] = R[1 + d] + (D2(u[d], d) + D(th - G[d][d], d)) / (ft(3) * Re)
        R[4] = R[4] - half * (D((E + two * p) * u[d] - two * V[d], d) + u[d] * D(E, d) + E * dU) + kappa * D2(Tm, d)
    return np.stack(R)


@pytest.mark.parametrize("order", [2, 4, 6, 8, 10, 12])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_residual_error_by_field(dtype, order):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    ft = np.float64 if dtype == "f64" else np.float32
    q = _state(order).astype(ft)
    ref = _plain(q, order, np.longdouble)
    plain = _plain(q, order, ft)
    s = sbli.Solver(SHAPE, order=order, dtype=dtype, **synth.TGV)
    qd = torch.from_numpy(q).cuda()
    if dtype == "f64":
        R = s.rhs(qd).cpu().numpy()
    else:
        # the residual that the stages use: so small a step leaves q as it is, and the second
        # stage has left dq = (1 + A_2) dt R
        dt = 1e-12
        dq = s.empty_state()
        s.rk3_step(qd, s.empty_state(), dq, dt, 1)
        R = dq.cpu().numpy().astype(np.float64) / (4.0 / 9.0 * float(np.float32(dt)))
    s.close()

    def rms(x):
        return np.sqrt(((x - ref) ** 2).mean(axis=(1, 2, 3))).astype(np.float64)

    ratio = rms(R) / rms(plain)
    print(dtype, order, "error over that of the plain formulation:", np.round(ratio, 3), flush=True)
    assert (ratio <= 1.0).all(), ratio
