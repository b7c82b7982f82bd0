"""Diagnostics with work items of every length (one plane, a few, a short last item) against the
FP64 oracle; 1e-12 relative, the bound of the other diagnostics tests."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,order", [((9, 9, 9), 4), ((32, 32, 32), 4), ((33, 18, 140), 8), ((100, 70, 61), 2),
                                         ((130, 64, 50), 12)])
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1)])
def test_diagnostics_match_oracle(oracle_mod, shape, order, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    q0 = synth.random_conservative_state(shape, seed=order, mom=0.3)
    s = sbli.Solver(shape, order=order, bc=bc, **synth.TGV)
    d, code = s.diagnostics(torch.from_numpy(q0).cuda(), check=False)
    assert code == 0
    ref, _ = oracle.diagnostics(q0, oracle.Params(n=shape, order=order, bc=bc, **synth.TGV))
    got = np.array([d[k] for k in ("Ek", "enstrophy", "rho", "rhou", "rhov", "rhow", "rhoE")])
    assert np.abs(got[:2] - ref[:2]).max() <= 1e-12 * np.abs(ref[:2]).max()
    assert np.abs(got[2:] - ref[2:]).max() <= 1e-12 * np.abs(ref[2:]).max()
