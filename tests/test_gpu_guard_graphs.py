"""Guard calls captured from one network, on terms, flags and counters of their own, replayed
beside each other on two streams and beside an eager call: every verdict is that of its own term."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 64])
def test_guards_of_one_network_beside_each_other(n):
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a HIP device")
    from paper_1609_01277_amd import closure
    own = torch.cuda.Stream()
    streams = [torch.cuda.Stream() for _ in range(2)]
    net = closure.ClosureNet(n, 1, stream=own)
    stats = np.zeros(35, np.float32)
    stats[5:10] = stats[15:20] = stats[20:25] = 1.0
    net.set_stats(stats)
    good = torch.full((5, n ** 3), 0.5, device="cuda")
    bad = good.clone()
    bad[4, n ** 3 - 1] = 2.0
    jobs = [dict(c=c, flag=torch.full((1,), 7, dtype=torch.int32, device="cuda"),
                 cnt=torch.zeros(2, dtype=torch.int32, device="cuda")) for c in (good, bad, good)]
    torch.cuda.synchronize()
    graphs = []
    for j in jobs[:2]:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=own):
            for _ in range(20):
                net.guard(j["c"], j["flag"], j["cnt"])
        graphs.append(g)
    for rep in range(1, 6):
        for g, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                g.replay()
        for _ in range(20):
            net.guard(jobs[2]["c"], jobs[2]["flag"], jobs[2]["cnt"])
        torch.cuda.synchronize()
        assert [j["flag"].item() for j in jobs] == [1, 0, 1]
        assert [j["cnt"].tolist() for j in jobs] == [[20 * rep, 0], [0, 20 * rep], [20 * rep, 0]]
    net.close()
