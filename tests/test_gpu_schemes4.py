"""GPU tests of the two ways that k = 4 is counted by default: core reuse for
small inputs and subgraph copies for the rest and for calls of several sizes.
Both sides of the line between them through every entry point, the copies on
small graphs (as one of two sizes), in batches and in undirected censuses large
enough for them, and the core-reuse kernel under its placement limits."""
import ctypes

import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_copies import clique, theta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    assert pm.lib().motif_init() == 0
    return pm


def exactly(n, m, seed):
    """m arcs of a power-law graph, with rows out of order."""
    g = gg.chung_lu(n, m, 2.3, 2.4, 0.2, seed=seed)
    assert g.m == m
    rng = np.random.default_rng(seed)
    idx = g.out_idx.copy()
    for v in range(n):
        a, b = int(g.out_off[v]), int(g.out_off[v + 1])
        idx[a:b] = rng.permutation(idx[a:b])
    return g, idx


@pytest.mark.parametrize("n,m", [(700, 5120), (700, 5121), (5120, 3000), (5121, 3000), (90, 1000), (3, 2)])
def test_line_of_one_graph(pm, n, m):
    import torch
    g, idx = exactly(n, m, n + m) if n > 3 else (gg.from_arcs(3, [(0, 1), (2, 1)]), np.asarray([1, 1], np.int32))
    print(f"[case] k = 4 either way n={n} m={m}", flush=True)
    want = oracle.method_census(g, 4)
    off_t, idx_t = pm.to_device(g.out_off, idx)
    io, ii = pm.to_device(*g.in_csr())
    assert np.array_equal(pm.census(off_t, idx_t, n, 4), want)
    assert np.array_equal(pm.census(off_t, idx_t, n, 4, io, ii), want)
    h3, h4 = pm.census_multi(off_t, idx_t, n, (3, 4))
    assert np.array_equal(h4, want) and np.array_equal(h3, oracle.method_census(g, 3))
    assert np.array_equal(pm.census_multi(off_t, idx_t, n, (4,), io, ii)[0], want)
    hist = torch.empty(199, dtype=torch.int64, device="cuda")
    status = torch.empty(1, dtype=torch.int32, device="cuda")
    pm.census_async(off_t, idx_t, n, 4, hist, status)
    torch.cuda.synchronize()
    assert status.item() == 0 and np.array_equal(hist.cpu().numpy().view(np.uint64), want)
    hist.fill_(3)
    rc = pm.lib().motif_census_noalloc(ctypes.c_void_p(off_t.data_ptr()), ctypes.c_void_p(idx_t.data_ptr()), None, None,
                                       n, m, 4, ctypes.c_void_p(hist.data_ptr()), None)
    assert rc == 0 and np.array_equal(hist.cpu().numpy().view(np.uint64), want)
    plan = pm.BatchPlan([(off_t, idx_t, n)], 4)
    assert np.array_equal(plan.hists()[0], want)
    plan.close()
    with pm.Server(512 << 20, 2) as srv:
        t = srv.submit(g.out_off, idx, n, 4)
        assert np.array_equal(srv.wait(t), want)
    und = oracle.census_undirected(g, 4) if n <= 700 and m <= 2000 else None
    if und is not None:
        assert np.array_equal(pm.census_undirected(off_t, idx_t, n, 4), und)


@pytest.mark.parametrize("m", [1792, 1793])  # eight graphs: 14,336 arcs and a few more
def test_line_of_a_batch(pm, m):
    gs = [exactly(400, m, 10 * m + i)[0] for i in range(8)]
    print(f"[case] batch k = 4 either way m={m}", flush=True)
    dev = [(*pm.to_device(g.out_off, g.out_idx), g.n) for g in gs]
    h = pm.census_batch(dev, 4)
    plan = pm.BatchPlan(dev, 4)
    for rep in range(2):
        assert np.array_equal(plan.hists(), h)
        plan.run()
    plan.close()
    for i, g in enumerate(gs):
        assert np.array_equal(h[i], oracle.method_census(g, 4)), i


@pytest.mark.parametrize("g", [clique(n, np.random.default_rng(n)) for n in (4, 17, 18, 41, 42, 65, 66)] +
                         [theta(n, np.random.default_rng(n)) for n in (2, 48, 49, 127, 128, 192, 193, 1000, 1001)],
                         ids=lambda g: f"n{g.n}m{g.m}")
def test_copies_of_small_graphs(pm, g):
    print(f"[case] copies n={g.n} m={g.m}", flush=True)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    for got, k in zip(pm.census_multi(off, idx, g.n, (3, 4)), (3, 4)):
        assert np.array_equal(got, oracle.method_census(g, k)), k


@pytest.mark.parametrize("count", [30, 400])
def test_copies_in_batches(pm, count):
    rng = np.random.default_rng(count)
    gs = [gg.chung_lu(200, 700, 2.3, 2.3, 0.1, seed=i) for i in range(8)]
    gs += [clique(n, rng) for n in (5, 17, 30, 66)] + [theta(n, rng) for n in (49, 128, 193)] + [gg.from_arcs(3, [])]
    want = [oracle.method_census(g, 4) for g in gs]
    dev = [(*pm.to_device(g.out_off, g.out_idx), g.n) for g in gs]
    print(f"[case] copies in a batch of {count}", flush=True)
    h = pm.census_batch([dev[i % len(gs)] for i in range(count)], 4)
    for i in range(count):
        assert np.array_equal(h[i], want[i % len(gs)]), i


def test_copies_undirected(pm):
    g = gg.chung_lu(1500, 6000, 2.4, 2.4, 0.0, seed=4)
    both = gg.from_arcs(g.n, np.unique(np.concatenate([g.arcs(), g.arcs()[:, ::-1]]), axis=0))
    print("[case] undirected by copies", flush=True)
    d = oracle.method_census(both, 4)
    want = np.zeros(6, np.uint64)
    for c in np.flatnonzero(d):
        want[pm.class_undirected(4, int(c))] += d[c]
    assert np.array_equal(pm.census_undirected(*pm.to_device(g.out_off, g.out_idx), g.n, 4), want)


def test_core_reuse_placement(pm):
    graphs = [gg.chung_lu(600, 4800, 2.1, 2.2, 0.2, seed=31), clique(66, np.random.default_rng(1)),
              theta(1200, np.random.default_rng(2)), gg.star(1500, 1200, 700)]
    want = [oracle.method_census(g, 4) for g in graphs]
    dev = [(*pm.to_device(g.out_off, g.out_idx), g.n) for g in graphs]
    saved = pm.get_tuning(4)
    try:
        for block in (256, 512, 1024):
            for solo, light, tile in ((1, 1, 1), (16, 96, 7), (64, 256, 64)):
                print(f"[case] core reuse block={block} solo={solo} light={light} tile={tile}", flush=True)
                pm.set_tuning(4, block=block, solo_deg=solo, light_deg=light, tile=tile)
                for d, w in zip(dev, want):
                    assert np.array_equal(pm.census(*d, 4), w)
                h = pm.census_batch(dev[:2], 4)
                assert np.array_equal(h[0], want[0]) and np.array_equal(h[1], want[1])
    finally:
        pm.set_tuning(4, **saved)


def test_autotune_of_copies(pm):
    # parameters that the counting of copies doesn't read stay as they are
    g = gg.chung_lu(4000, 30000, 2.3, 2.4, 0.2, seed=4)
    dev = [(*pm.to_device(g.out_off, g.out_idx), g.n)]
    for k in (3, 4):
        saved = pm.get_tuning(k)
        try:
            print(f"[case] autotune by copies k={k}", flush=True)
            best = pm.autotune(dev, k)
            assert {f: v for f, v in best.items() if f != "heavy"} == {f: v for f, v in saved.items() if f != "heavy"}
            assert np.array_equal(pm.census(*dev[0], k), oracle.method_census(g, k))
        finally:
            pm.set_tuning(k, **saved)
