"""GPU tests of the census server's budget: a k = 4 request whose subgraph copies
take more room than the budget is counted by the reuse of cores where that fits,
and refused where neither does."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu
MB = 1 << 20


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


@pytest.mark.parametrize("n,m,budget", [(1000, 562341, 64 * MB)])
def test_dense_request_within_budget(pm, n, m, budget):
    rng = np.random.default_rng(n)
    code = rng.choice(n * (n - 1), m, replace=False)
    u, v = code // (n - 1), code % (n - 1)
    g = gg.from_arcs(n, np.c_[u, v + (v >= u)])
    fp = pm.request_footprint(g.n, g.m, 4)
    print(f"[case] n={n} m={m}: {fp / MB:.1f} MB, budget {budget / MB:.0f}", flush=True)
    assert fp > budget
    want = pm.census(*pm.to_device(g.out_off, g.out_idx), g.n, 4)
    with pm.Server(budget, max_inflight=2) as srv:
        ts = [srv.submit(g.out_off, g.out_idx, g.n, 4) for _ in range(3)]
        for t in ts:
            assert np.array_equal(srv.wait(t), want)
        assert srv.stats()["peak_bytes"] <= budget
    with pm.Server(2 * MB, max_inflight=1) as srv:
        with pytest.raises(pm.MotifError) as e:
            srv.submit(g.out_off, g.out_idx, g.n, 4)
        assert e.value.name == "ETOOBIG"
