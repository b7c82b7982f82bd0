"""The 8-channel convolutions take a quarter of the 32-channel one's products and write a quarter
(8 -> 8) or as much (5 -> 32) of its output: their time must say so.  (Reads of the staged points
that are not LDS instructions took half of the 32-channel form's time.)"""
import pytest

pytestmark = pytest.mark.gpu


def test_narrow_forms_take_their_share_of_the_time():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    n, batch = 64, 4
    P = n ** 3 * batch

    def us(f):
        f()
        best = 1e9
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                f()
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) * 50)
        return best

    t = {}
    for ci, co in ((32, 32), (8, 8), (5, 32)):
        cp, op = closure.sbli_conv3d_cpad(ci), closure.sbli_conv3d_cpad(co)
        x, dy = (torch.rand(P * c, device="cuda").bfloat16() for c in (cp, op))
        W, b = torch.rand(co * ci * 27, device="cuda"), torch.rand(32, device="cuda")
        Wf, Wb = (torch.zeros(32 * closure.sbli_conv3d_packed_width(c), device="cuda", dtype=torch.bfloat16) for c in (ci, co))
        closure.sbli_conv3d_pack(W, ci, co, Wf, Wb)
        pre, dx = torch.empty(P * 32, device="cuda"), torch.empty(P * 32, device="cuda")
        t[ci, co] = (us(lambda: closure.sbli_conv3d_fwd(x, ci, Wf, b, co, n, batch, closure.ACT_NONE, pre)),
                     us(lambda: closure.sbli_conv3d_bwd_data(dy, co, Wb, n, batch, None, dx)))
    print({k: "%.1f %.1f us" % v for k, v in t.items()}, flush=True)
    assert t[8, 8][0] <= 0.42 * t[32, 32][0]
    assert t[5, 32][0] <= 0.46 * t[32, 32][0]
    assert t[8, 8][1] <= 0.45 * t[32, 32][1]
