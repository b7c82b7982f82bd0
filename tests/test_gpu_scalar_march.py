"""Many steps of the scalar equation in one launch: one and two axes, a workgroup's field
(ring) and tiles, against the FP64 oracle at the sizes where the forms meet and at ragged ends."""
import numpy as np
import pytest

import oracle
from test_gpu_scalar import _mods, oracle_rhs

pytestmark = pytest.mark.gpu

CASES = [
    ((12, 1, 1), 12), ((65, 1, 1), 8), ((1, 511, 1), 2), ((512, 1, 1), 6), ((513, 1, 1), 12), ((1, 1, 1000), 8),
    ((16385, 1, 1), 4), ((82001, 1, 1), 10),                    # one axis: ring, tiles of 64 and of 320 points
    ((2, 2, 1), 2), ((12, 192, 1), 12), ((1, 48, 48), 4), ((37, 1, 29), 6),       # two axes: ring
    ((49, 48, 1), 2), ((1, 700, 13), 12), ((61, 1, 97), 4), ((301, 258, 1), 6),   # two axes: tiles
    ((11, 40, 1), 12), ((9, 8, 7), 4),                          # a launch a stage
]


@pytest.mark.parametrize("shape,order", CASES)
@pytest.mark.parametrize("with_source", [False, True])
def test_many_steps_match_oracle(oracle_mod, shape, order, with_source):
    """7 steps leave a remainder after every number of steps of a launch; 21 stages of some
    30 operations lose at most 21 * 30 * 2^-53 = 7e-14 relative to the field."""
    scalar, torch = _mods()
    length = tuple(0.1 * n if n > 1 else 1.0 for n in shape)
    c, k, dt, steps = (1.0, -0.5, 0.25), 0.75, 2e-4, 7
    P = shape[0] * shape[1] * shape[2]
    rng = np.random.default_rng(P + order)
    phi0 = rng.standard_normal(P)
    S = rng.standard_normal(P) if with_source else None
    ref = oracle.rk3_generic(phi0, dt, steps, lambda y: oracle_rhs(y, shape, order, length, c, k, S))
    p = scalar.params(shape, length, order, c, k)
    phi = torch.from_numpy(phi0).cuda()
    Sd = None if S is None else torch.from_numpy(S).cuda()
    scalar.sbli_scalar_rk3(p, phi, torch.empty_like(phi), torch.empty_like(phi), Sd, dt, steps)
    assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
