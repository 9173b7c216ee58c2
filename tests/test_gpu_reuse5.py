"""GPU tests of the k = 5 core-reuse kernel, which counts batches, asynchronous
calls and the graphs that the subgraph copies leave out: its blocks, tiles and
grids, the placement limit of its light units, the sub-chunks of light partners,
and the W rows kept from call to call.  Through batches, which always take it."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_census import _partner_fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


@pytest.fixture
def tuned(pm):
    saved = pm.get_tuning(5)
    yield lambda **kw: pm.set_tuning(5, **kw)
    pm.set_tuning(5, **saved)


def reuse5(pm, g, stream=None):
    off, idx = pm.to_device(g.out_off, g.out_idx)
    return pm.census_batch([(off, idx, g.n)], 5, stream=stream)[0]


def test_blocks_tiles_grids(pm, tuned):
    g = gg.chung_lu(700, 3000, 2.2, 2.3, 0.1, seed=90)
    want = oracle.method_census(g, 5)
    for block in (512, 1024):
        for tile in (1, 7, 64):
            for gpc in (1, 3):
                print(f"[case] block={block} tile={tile} gpc={gpc}", flush=True)
                tuned(block=block, tile=tile, grid_per_cu=gpc, heavy=1)
                assert np.array_equal(reuse5(pm, g), want)


def test_light_limit(pm, tuned):
    g = gg.chung_lu(700, 3500, 2.2, 2.5, 0.1, seed=32)
    want = oracle.method_census(g, 5)
    for light5 in (1, 64, 767):
        print(f"[case] light5={light5}", flush=True)
        tuned(light5=light5)
        assert np.array_equal(reuse5(pm, g), want)


def test_light_subchunks(pm, tuned):
    g = _partner_fan()
    for name, x in (("partner fan", g), ("relabelled", gg.relabel(g, seed=6))):
        print(f"[case] {name} n={x.n}", flush=True)
        assert np.array_equal(reuse5(pm, x), oracle.method_census(x, 5))
    g = _partner_fan(n_part=12, d_part=300, d_a=400, seed=7)
    print(f"[case] wide partner fan n={g.n}", flush=True)
    a = reuse5(pm, g)
    tuned(heavy=2)
    assert np.array_equal(a, reuse5(pm, g)) and a.sum() > 0


def test_w_rows_kept(pm):
    import torch
    s = torch.cuda.Stream()
    graphs = [gg.chung_lu(2000, 9000, 2.1, 2.1, 0.2, seed=91), gg.chung_lu(800, 4000, 2.2, 2.3, 0.1, seed=92)]
    want = [oracle.method_census(g, 5) for g in graphs]
    for i in (0, 1, 0, 1, 1, 0):
        print(f"[case] W rows n={graphs[i].n}", flush=True)
        assert np.array_equal(reuse5(pm, graphs[i], s), want[i])
