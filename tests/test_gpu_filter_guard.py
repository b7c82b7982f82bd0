"""Edges of the box filter's row form and of the many-workgroup closure guard."""
import numpy as np
import pytest

import synth
from oracle import nn

pytestmark = pytest.mark.gpu
U = 2.0 ** -24   # unit roundoff of the FP32 output


def _mods():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    return closure, torch


# nc = nf / ratio: below, at and beyond a 64-lane row; rows and planes left over by a workgroup's
# 4 x 4; ratio 6 and an odd element offset take the pointwise form
@pytest.mark.parametrize("nf,ratio,offset", [(4, 2, 0), (34, 2, 0), (128, 2, 0), (130, 2, 0), (12, 4, 0), (76, 4, 0),
                                             (260, 4, 0), (16, 8, 0), (72, 8, 0), (36, 6, 0), (76, 4, 1)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_box_filter_edges_match_oracle(nf, ratio, offset, dtype):
    closure, torch = _mods()
    nfields = 5 if nf < 200 else 1
    f = synth.random_conservative_state(nf, seed=nf + ratio)[:nfields]
    t = torch.float64 if dtype == "f64" else torch.float32
    buf = torch.empty(nfields * nf ** 3 + offset, dtype=t, device="cuda")
    fine = buf[offset:].view(nfields, nf, nf, nf)
    fine.copy_(torch.from_numpy(np.ascontiguousarray(f)))
    nc = nf // ratio
    src = fine.cpu().numpy().astype(np.float64)
    ref = nn.box_filter(src, ratio)
    # FP64 sums of (ratio + 1)^3 weighted values, three nested sums: below 4 (ratio + 3) 2^-53 of the
    # largest value; then one rounding to FP32
    tol = U * np.abs(ref) + 4 * (ratio + 3) * 2.0 ** -53 * np.abs(src).max()
    out = torch.empty((nfields, nc, nc, nc), dtype=torch.float32, device="cuda")
    closure.sbli_box_filter(fine, nf, nfields, ratio, out)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - ref) <= tol)
    c0 = np.random.default_rng(nf).standard_normal(ref.shape).astype(np.float32)
    out = torch.from_numpy(c0).cuda()
    closure.sbli_box_filter(fine, nf, nfields, ratio, out, subtract=True)
    got = out.cpu().numpy().astype(np.float64)
    want = ref - c0.astype(np.float64)
    assert np.all(np.abs(got - want) <= U * np.abs(want) + 4 * (ratio + 4) * 2.0 ** -53 * (np.abs(src).max() + 5.0))


@pytest.mark.parametrize("n", [32, 64])
def test_guard_finds_one_bad_value_anywhere(n):
    """One value beyond its own field's limit (or not finite) anywhere rejects; a value at the limit is
    accepted; verdict and counters stay right from call to call."""
    closure, torch = _mods()
    net = closure.ClosureNet(n, 1)
    st = np.ones(closure.N_STATS, dtype=np.float32)
    limits = (1.0, 2.0, 3.0, 4.0, 5.0)
    st[20:25] = limits
    net.set_stats(st)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(2, dtype=torch.int32, device="cuda")
    P = n ** 3
    c = torch.empty((5, P), dtype=torch.float32, device="cuda")
    for f in range(5):
        c[f] = limits[f]
    accepted = rejected = 0
    for f in range(5):
        for p in (0, 1, 4095, 4096, P // 2, P - 1):
            for bad in (limits[f] * 1.0001, -limits[f] * 1.0001, float("nan"), float("inf")):
                c[f, p] = bad
                net.guard(c, flag, cnt)
                rejected += 1
                assert flag.item() == 0 and cnt.tolist() == [accepted, rejected], (f, p, bad)
                c[f, p] = -limits[f]
                net.guard(c, flag, cnt)
                accepted += 1
                assert flag.item() == 1 and cnt.tolist() == [accepted, rejected], (f, p)
    net.close()
