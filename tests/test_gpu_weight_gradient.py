"""The weight-gradient kernel's operand choices and work split against the oracle, every element:
both tensors narrow (8 channels), one of them, none; channel counts below the padded ones; one
plane per workgroup, several, and runs that cross from one column of points to the next."""
import numpy as np
import pytest

from oracle import nn

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("n,batch,cin,cout", [
    (32, 1, 5, 32), (32, 1, 32, 5), (32, 3, 20, 32), (32, 1, 9, 12), (32, 2, 8, 3), (64, 1, 32, 8), (64, 1, 32, 32),
    (64, 2, 5, 5), (96, 1, 5, 9)])
def test_weight_gradient_matches_oracle(n, batch, cin, cout):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    P = n ** 3
    g = torch.Generator().manual_seed(n * 1000 + cin * 40 + cout)
    pad = lambda c: 8 if c <= 8 else 32   # noqa: E731
    x = torch.zeros((batch, P, pad(cin)), dtype=torch.bfloat16)
    d = torch.zeros((batch, P, pad(cout)), dtype=torch.bfloat16)
    x[..., :cin] = torch.randn((batch, P, cin), generator=g).to(torch.bfloat16)
    d[..., :cout] = torch.randn((batch, P, cout), generator=g).to(torch.bfloat16)
    work = torch.full((closure.sbli_conv3d_bwd_weight_work_bytes(cin) // 4,), float("nan"), device="cuda")
    dW = torch.empty((cout, cin, 27), device="cuda")
    db = torch.empty(cout, device="cuda")
    closure.sbli_conv3d_bwd_weight(x.cuda(), cin, d.cuda(), cout, n, batch, dW, db, work)
    first = dW.clone()
    closure.sbli_conv3d_bwd_weight(x.cuda(), cin, d.cuda(), cout, n, batch, dW, db, work)
    assert torch.equal(first, dW)         # the sum's order is fixed
    pl = lambda a, c: a.float().numpy().reshape(batch, n, n, n, -1)[..., :c].transpose(0, 4, 1, 2, 3).astype(np.float64)  # noqa: E731, E501
    xs, ds = pl(x, cin), pl(d, cout)
    rW, _ = nn.conv3d_bwd_weight(xs, ds)
    aW, _ = nn.conv3d_bwd_weight(np.abs(xs), np.abs(ds))
    # additions along a chain: 256 points a plane in 16-point products, then the partials in four
    # interleaved chains; a full unit each (an accumulator may truncate), twice for safety
    planes = batch * n * (n // 8) * (n // 32)
    per = -(-planes // 512)
    depth = per * 256 + 512 // 4 + 3
    err = np.abs(dW.cpu().numpy().reshape(cout, cin, 3, 3, 3).astype(np.float64) - rW)
    assert np.all(err <= 2 * (depth + 2) * U * aW), err.max()
