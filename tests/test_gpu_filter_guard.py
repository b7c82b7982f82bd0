"""Edges of the many-workgroup closure guard."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _mods():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    return closure, torch


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
