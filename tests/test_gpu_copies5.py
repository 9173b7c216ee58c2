"""GPU tests of the k = 5 census from typed subgraph copies at the edges of its
tables: links of an entry (8 or more, 256 or more), vertices adjacent to a
triangle (64), rows of 1,024 and degrees of 127 around them, wedge hashes, and
graphs that it leaves to the per-core scan.  Counts are whole numbers and
compared exactly with the CPU oracle."""
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


def from_edges(n, edges, seed, r=0.3):
    """Edges (pairs) with random directions, a share r of them both ways, ids permuted."""
    rng = np.random.default_rng(seed)
    e = np.asarray(edges, np.int64)
    e = np.unique(np.c_[e.min(1), e.max(1)], axis=0)
    e = rng.permutation(n)[e]
    t = rng.random(len(e))
    fw, bw = t < (1 + r) / 2, t >= (1 - r) / 2
    return gg.from_arcs(n, np.concatenate([e[fw], e[bw][:, ::-1]]))


def check(pm, g, label):
    print(f"[case] {label} n={g.n} m={g.m}", flush=True)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    want = oracle.census(g, 5) if g.m <= 300 else oracle.method_census(g, 5)
    assert np.array_equal(pm.census(off, idx, g.n, 5), want), label


@pytest.mark.parametrize("seed", range(12))
def test_small(pm, seed):
    rng = np.random.default_rng(seed)
    n = int(rng.integers(5, 13))
    check(pm, gg.random_small(n, float(rng.uniform(0.05, 0.6)), float(rng.uniform(0, 1)), seed=seed), "small")


@pytest.mark.parametrize("c,n", [(5, 12), (10, 24), (11, 24), (66, 150), (67, 150), (70, 71)])
def test_clique_with_tails(pm, c, n):
    """A clique of c and a path through the other vertices hung on it (70 of 71: nearly all pairs joined)."""
    a, b = np.triu_indices(c, 1)
    tail = [(i, i + 1) for i in range(c - 1, n - 1)] + [(i, i % c) for i in range(c, n, 3)]
    check(pm, from_edges(n, np.r_[np.c_[a, b], np.asarray(tail).reshape(-1, 2)], c), "clique")


@pytest.mark.parametrize("d", [126, 127, 128, 300])
def test_book(pm, d):
    """An edge with d thirds, a path through the thirds and pendants."""
    t = 2 + np.arange(d)
    e = [(0, 1)] + [(0, x) for x in t] + [(1, x) for x in t] + [(x, x + 1) for x in t[:-1]]
    e += [(x, d + 2 + k) for k, x in enumerate(t[::5])]
    check(pm, from_edges(2 + d + len(t[::5]), e, d), "book")


@pytest.mark.parametrize("d", [1022, 1023, 1024, 1100])
def test_hub_over_a_ring(pm, d):
    """A hub joined to a ring of d and, with 40 of the ring, to a second hub."""
    ring = 2 + np.arange(d)
    e = [(0, x) for x in ring] + [(x, 2 + (x - 1) % d) for x in ring] + [(0, 1)] + [(1, x) for x in ring[::d // 40]]
    check(pm, from_edges(2 + d, e, d), "hub")


@pytest.mark.parametrize("mids", [2, 96, 127, 128, 400])
def test_theta(pm, mids):
    e = [(0, 2 + i) for i in range(mids)] + [(1, 2 + i) for i in range(mids)] + [(2 + i, 2 + mids + i % 7) for i in range(mids)]
    check(pm, from_edges(2 + mids + 7, e, mids), "theta")


@pytest.mark.parametrize("n,m,go,gi,r,seed", [(700, 3000, 2.2, 2.3, 0.1, 90), (4000, 20000, 2.4, 2.4, 0.1, 4),
                                              (3000, 24000, 2.1, 2.1, 0.2, 2), (13000, 30000, 2.1, 2.4, 0.0, 7)])
def test_power_law(pm, n, m, go, gi, r, seed):
    check(pm, gg.chung_lu(n, m, go, gi, r, seed=seed), "power law")


def test_all_sizes_share_a_call(pm):
    g = gg.chung_lu(900, 5000, 2.3, 2.3, 0.2, seed=3)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    for ks in ((3, 4, 5), (5, 3), (4, 5)):
        got = pm.census_multi(off, idx, g.n, ks)
        for i, k in enumerate(ks):
            assert np.array_equal(got[i], oracle.method_census(g, k)), (ks, k)
