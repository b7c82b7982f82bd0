"""The device memory that sbli_init takes without being asked (the staged form's scratch, the
default of orders 6 and 8) is bounded for all contexts together, and given back."""
import gc

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,order,n", [("f64", 8, 256), ("f64", 6, 256), ("f32", 8, 320)])
def test_many_contexts_keep_to_the_share(dtype, order, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    import paper_1609_01277_amd as sbli
    scratch = 6 * n ** 3 * (8 if dtype == "f64" else 4)
    gc.collect()                                           # contexts that earlier tests left
    torch.cuda.synchronize()
    free0, total = torch.cuda.mem_get_info()
    share = total // 64
    count = share // scratch + 3
    small = 16 << 20                                       # a context's other scratch, rounded up by the allocator
    for _ in range(2):                                     # the second time after everything was given back
        solvers = [sbli.Solver(n, order=order, dtype=dtype, **synth.TGV) for _ in range(count)]
        taken = free0 - torch.cuda.mem_get_info()[0]
        staged = [s.get_tuning()[0] == len(s.variants()) - 1 for s in solvers]
        for s in solvers:
            s.close()
        assert staged[0] and not any(staged[share // scratch:])
        assert taken <= share + count * small, (taken, share)
    assert free0 - torch.cuda.mem_get_info()[0] <= small
