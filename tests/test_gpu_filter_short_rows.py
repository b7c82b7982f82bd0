"""Box filter on many fields of short rows: an aligned base must not be slower than one that is not
(which always takes the pointwise form), and both give the same bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,ratio,nc", [("f64", 2, 8), ("f64", 2, 16), ("f64", 4, 6), ("f64", 4, 8), ("f64", 8, 6),
                                            ("f32", 2, 16), ("f32", 4, 6), ("f32", 8, 6), ("f64", 4, 12), ("f64", 8, 8),
                                            ("f64", 2, 20), ("f32", 4, 10), ("f32", 8, 7), ("f64", 8, 10)])
def test_short_rows_of_many_fields(dtype, ratio, nc):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    nf, fields = nc * ratio, 320
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(nc)
    buf = torch.rand(fields * nf ** 3 + 1, dtype=dt, device="cuda", generator=g)
    aligned = buf[1:].clone()
    out = [torch.empty(fields * nc ** 3, dtype=torch.float32, device="cuda") for _ in range(2)]

    def us(x, y):
        closure.sbli_box_filter(x, nf, fields, ratio, y)
        best = 1e9
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                closure.sbli_box_filter(x, nf, fields, ratio, y)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) * 50)
        return best

    t = us(aligned, out[0]), us(buf[1:], out[1])
    print(dtype, ratio, nc, "us aligned %.1f, not aligned %.1f" % t, flush=True)
    assert torch.equal(out[0], out[1])
    assert t[0] <= 1.2 * t[1] + 1.0
