"""GPU tests of the censuses from typed subgraph copies (k = 3, 4) at the edges
of their tiers: the higher neighbours of a vertex (16, 64, 128, 256), the visits
and lower neighbours behind a wedge table (96, 384, 3,072 and 127, 1,000), the
id blocks of 12,288, more hubs than one pass holds, and batches in which only a
few vertices reach a tier.  Counts are whole numbers and compared exactly with
the per-anchor method on the CPU."""
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


def from_edges(n, a, b, rng, r=0.3, shuffle=True):
    """Undirected edges a - b with random directions, a share r of them both ways, and ids permuted."""
    a, b = np.asarray(a, np.int64), np.asarray(b, np.int64)
    if shuffle:
        ids = rng.permutation(n)
        a, b = ids[a], ids[b]
    t = rng.random(len(a))
    fw, bw = t < (1 + r) / 2, t >= (1 - r) / 2
    return gg.from_arcs(n, np.concatenate([np.c_[a[fw], b[fw]], np.c_[b[bw], a[bw]]]))


def clique(n, rng):
    a, b = np.triu_indices(n, 1)
    return from_edges(n, a, b, rng)


def theta(mids, rng, far=4):
    """Two poles joined by `mids` middle vertices, and some pendants on the first pole."""
    n = 2 + mids + far
    a = np.concatenate([np.zeros(mids), np.ones(mids), np.zeros(far)])
    b = np.concatenate([2 + np.arange(mids), 2 + np.arange(mids), 2 + mids + np.arange(far)])
    return from_edges(n, a, b, rng)


def check(pm, g, k, label):
    print(f"[case] {label} k={k} n={g.n} m={g.m}", flush=True)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    assert np.array_equal(pm.census(off, idx, g.n, k), oracle.method_census(g, k)), label


@pytest.mark.parametrize("k", [3, 4])
@pytest.mark.parametrize("n", [17, 18, 65, 66, 129, 130, 257, 259])
def test_clique(pm, n, k):
    check(pm, clique(n, np.random.default_rng(n)), k, "clique")


@pytest.mark.parametrize("mids", [48, 49, 127, 128, 192, 193, 1000, 1001, 1600])
def test_theta(pm, mids):
    check(pm, theta(mids, np.random.default_rng(mids)), 4, "theta")


@pytest.mark.parametrize("each,pole", [(29, 100), (30, 100), (31, 100), (29, 106), (28, 127), (28, 128)])
def test_visits(pm, each, pole):
    """A pole over `pole` middle vertices of `each` + 1 neighbours among 150 far ones: visits around 3,072."""
    rng = np.random.default_rng(each * pole)
    far = np.concatenate([rng.choice(150, each, replace=False) for _ in range(pole)])
    a = np.concatenate([np.zeros(pole), np.repeat(1 + np.arange(pole), each)])
    b = np.concatenate([1 + np.arange(pole), 1 + pole + far])
    check(pm, from_edges(1 + pole + 150, a, b, rng), 4, "visits")


@pytest.mark.parametrize("n,m", [(12_288, 30_000), (12_289, 34_000), (30_000, 60_000)])
def test_blocks(pm, n, m):
    """Wedges across the id blocks, with and without blocks cut by entries: two poles over 2,500 middles and noise."""
    rng = np.random.default_rng(n)
    a = np.concatenate([np.zeros(2500), np.full(2500, n - 1), rng.integers(0, n, m)])
    b = np.concatenate([1 + np.arange(2500), 1 + np.arange(2500), rng.integers(0, n, m)])
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    e = np.unique((lo * n + hi)[lo != hi].astype(np.int64))
    check(pm, from_edges(n, e // n, e % n, rng, shuffle=False), 4, "blocks")


def test_many_hubs(pm):
    """A complete bipartite graph with 1,100 vertices of degree 130: more hubs than one pass holds."""
    a, b = np.meshgrid(np.arange(130), 130 + np.arange(1100), indexing="ij")
    check(pm, from_edges(1230, a.ravel(), b.ravel(), np.random.default_rng(0)), 4, "hubs")


@pytest.mark.parametrize("k", [3, 4])
@pytest.mark.parametrize("few", [1, 3])
def test_batch_with_few_in_a_tier(pm, k, few):
    rng = np.random.default_rng(few)
    graphs = [gg.chung_lu(300, 900, 2.3, 2.3, 0.1, seed=i) for i in range(40)]
    for i in range(few):
        graphs.insert(7 * i + 5, clique(20 + 60 * i, rng))
        graphs.insert(7 * i + 9, theta(60 + 70 * i, rng))
    graphs.insert(2, gg.from_arcs(0, []))
    print(f"[case] batch k={k} graphs={len(graphs)}", flush=True)
    h = pm.census_batch([(*pm.to_device(g.out_off, g.out_idx), g.n) for g in graphs], k)
    for i, g in enumerate(graphs):
        assert np.array_equal(h[i], oracle.method_census(g, k)), f"graph {i}"
