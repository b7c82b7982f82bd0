"""The box filter's row form with 1, 2 and 4 output planes a workgroup: bit for bit the pointwise
form, which an odd element offset selects."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,ratio", [(36, 2), (130, 2), (200, 2), (72, 4), (164, 4), (256, 4), (144, 8), (248, 8),
                                      (512, 8)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("subtract", [False, True])
def test_rows_equal_pointwise(nf, ratio, dtype, subtract):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    t = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(nf + ratio)
    n = 5 * nf ** 3
    fine = torch.randn(n, generator=g, device="cuda", dtype=t)
    odd = torch.empty(n + 1, device="cuda", dtype=t)[1:]
    odd.copy_(fine)
    c0 = torch.randn((5,) + (nf // ratio,) * 3, generator=g, device="cuda")
    a, b = c0.clone(), c0.clone()
    closure.sbli_box_filter(fine, nf, 5, ratio, a, subtract=subtract)
    closure.sbli_box_filter(odd, nf, 5, ratio, b, subtract=subtract)
    assert torch.isfinite(a).all() and torch.equal(a, b)
