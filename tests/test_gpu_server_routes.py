"""GPU tests of how the census server counts k = 4 requests: a server of one
request in flight as a census call does (small graphs by the reuse of cores), one
of several by subgraph copies, seen by the bytes that a request holds."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


@pytest.mark.parametrize("n,m,reuse", [(1000, 4000, True), (3000, 20000, False)])
def test_route_by_requests_in_flight(pm, n, m, reuse):
    g = gg.chung_lu(n, m, 2.4, 2.4, 0.1, seed=m)
    want = oracle.method_census(g, 4)
    fp = pm.request_footprint(g.n, g.m, 4)
    for workers in (1, 2):
        print(f"[case] n={n} m={g.m} workers={workers}", flush=True)
        with pm.Server(1 << 30, max_inflight=workers) as srv:
            assert np.array_equal(srv.wait(srv.submit(g.out_off, g.out_idx, g.n, 4)), want)
            peak = srv.stats()["peak_bytes"]
        assert peak < fp if reuse and workers > 1 else peak == fp
