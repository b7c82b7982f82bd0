"""Forward and backward-data convolutions against FP64 at the sizes where the staging differs:
one, two and three x tiles (the end points of a row wrap), 8 and 32 channels."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(32, 2), (64, 1), (96, 1)])
@pytest.mark.parametrize("cin,cout", [(5, 32), (32, 5)])
def test_conv_matches_fp64(n, batch, cin, cout):
    """FP32 sums of 27 cin exact products of BF16 numbers: off by at most 27 cin 2^-24 of the
    sum of their magnitudes."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    g = torch.Generator().manual_seed(n + cin)
    cpad = closure.sbli_conv3d_cpad(cin)
    x = torch.zeros((batch, n ** 3, cpad), dtype=torch.bfloat16)
    x[..., :cin] = torch.randn((batch, n ** 3, cin), generator=g).to(torch.bfloat16)
    W = torch.randn((cout, cin, 27), generator=g).to(torch.bfloat16).float()
    Wf = torch.zeros((32, closure.sbli_conv3d_packed_width(cin)), dtype=torch.bfloat16, device="cuda")
    Wb = torch.zeros((32, closure.sbli_conv3d_packed_width(cout)), dtype=torch.bfloat16, device="cuda")
    closure.sbli_conv3d_pack(W.cuda(), cin, cout, Wf, Wb)
    opad = closure.sbli_conv3d_cpad(cout)
    y = torch.zeros((batch, n ** 3, opad), device="cuda")
    closure.sbli_conv3d_fwd(x.cuda(), cin, Wf, torch.zeros(cout, device="cuda"), cout, n, batch, closure.ACT_NONE, y)
    got = y.cpu().double()[..., :cout]
    x3 = x.double()[..., :cin].reshape(batch, n, n, n, cin).permute(0, 4, 1, 2, 3)
    pad = torch.nn.functional.pad(x3, (1,) * 6, mode="circular")
    w3 = W.double().reshape(cout, cin, 3, 3, 3)
    conv = lambda a, w: torch.nn.functional.conv3d(a, w).permute(0, 2, 3, 4, 1).reshape(batch, n ** 3, cout)
    ref, mag = conv(pad, w3), conv(pad.abs(), w3.abs())
    assert bool(((got - ref).abs() <= 27 * cin * 2.0 ** -24 * mag).all())
    if cin == 32:
        dx = torch.empty((batch, n ** 3, 32), device="cuda")
        d = torch.zeros((batch, n ** 3, opad), dtype=torch.bfloat16)
        d[..., :cout] = torch.randn((batch, n ** 3, cout), generator=g).to(torch.bfloat16)
        closure.sbli_conv3d_bwd_data(d.cuda(), cout, Wb, n, batch, None, dx)
        d3 = d.double()[..., :cout].reshape(batch, n, n, n, cout).permute(0, 4, 1, 2, 3)
        pad = torch.nn.functional.pad(d3, (1,) * 6, mode="circular")
        wt = w3.flip(2, 3, 4).transpose(0, 1).contiguous()
        conv = lambda a, w: torch.nn.functional.conv3d(a, w).permute(0, 2, 3, 4, 1).reshape(batch, n ** 3, 32)
        ref, mag = conv(pad, wt), conv(pad.abs(), wt.abs())
        assert bool(((dx.cpu().double() - ref).abs() <= 27 * cout * 2.0 ** -24 * mag).all())
