"""GPU tests of graphs that the k = 5 census by subgraph copies begins and then
leaves to the core-reuse kernel, having more triangles than its links have room
for: the graph built and the sizes 3 and 4 counted by then are used on.  Below
and above the number of arcs from which the wedges run beside the triangles."""
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


def _one_way(n, seed):
    """A third of all ordered pairs as arcs, none reciprocated: 0.3 n^3 / 6 triangles."""
    rng = np.random.default_rng(seed)
    a, b = np.triu_indices(n, 1)
    pick = rng.permutation(len(a))[:n * (n - 1) // 3]
    a, b, back = a[pick], b[pick], rng.random(len(pick)) < 0.5
    return gg.from_arcs(n, np.c_[np.where(back, b, a), np.where(back, a, b)])


def test_left_small(pm):
    g = _one_way(66, 1)
    adj = np.zeros((66, 66), np.int64)
    adj[tuple(g.arcs().T)] = 1
    adj |= adj.T
    links = int(np.trace(adj @ adj @ adj))  # six per triangle
    assert links > 48 * g.m + 4096 and 3 * g.m <= g.n * (g.n - 1)
    want = {k: oracle.method_census(g, k) for k in (3, 4, 5)}
    off, idx = pm.to_device(g.out_off, g.out_idx)
    io, ii = pm.to_device(*g.in_csr())
    both = gg.from_arcs(66, np.unique(np.concatenate([g.arcs(), g.arcs()[:, ::-1]]), axis=0))
    und = np.zeros(21, np.uint64)
    d = oracle.method_census(both, 5)
    for c in np.flatnonzero(d):
        und[pm.class_undirected(5, int(c))] += d[c]
    other = gg.chung_lu(500, 2500, 2.3, 2.3, 0.2, seed=1)
    oo, oi = pm.to_device(other.out_off, other.out_idx)
    want_other = oracle.method_census(other, 5)
    for rep in range(3):
        print(f"[case] left to the cores m={g.m} round {rep}", flush=True)
        assert np.array_equal(pm.census(off, idx, g.n, 5), want[5])
        assert np.array_equal(pm.census(off, idx, g.n, 5, io, ii), want[5])
        for ks in ((3, 4, 5), (5, 3), (4, 5), (5,)):
            for got, k in zip(pm.census_multi(off, idx, g.n, ks, io, ii), ks):
                assert np.array_equal(got, want[k]), (ks, k)
        assert np.array_equal(pm.census_undirected(off, idx, g.n, 5), und)
        assert np.array_equal(pm.census(oo, oi, other.n, 5), want_other)
        assert np.array_equal(pm.census_batch([(off, idx, g.n), (oo, oi, other.n)], 5)[0], want[5])
    with pm.Server(256 << 20, 2) as srv:
        for t in [srv.submit(g.out_off, g.out_idx, g.n, 5) for _ in range(4)]:
            assert np.array_equal(srv.wait(t), want[5])


def test_left_large(pm):
    g = _one_way(330, 2)
    assert g.m >= 32768
    off, idx = pm.to_device(g.out_off, g.out_idx)
    saved = pm.get_tuning(5)
    try:
        print(f"[case] per anchor m={g.m}", flush=True)
        pm.set_tuning(5, heavy=2)
        want = pm.census(off, idx, g.n, 5)
    finally:
        pm.set_tuning(5, **saved)
    print(f"[case] left to the cores m={g.m}", flush=True)
    h3, h4, h5 = pm.census_multi(off, idx, g.n, (3, 4, 5))
    assert np.array_equal(h5, want)
    assert np.array_equal(h3, oracle.method_census(g, 3)) and np.array_equal(h4, oracle.method_census(g, 4))
    assert np.array_equal(pm.census(off, idx, g.n, 5), want)
