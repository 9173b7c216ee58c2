"""GPU test of the k = 4 census where the adjacency slices of large dense
neighbourhoods are fewer than workgroups (10^6 arcs): vertices on both sides of
256 higher neighbours, which are launches of their own there."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_copies import clique

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


def test_few_slices(pm):
    rng = np.random.default_rng(4)
    dense = gg.disjoint_union(clique(330, rng), clique(270, rng))
    pairs = np.arange(1_900_000).reshape(-1, 2)
    g = gg.disjoint_union(dense, gg.from_arcs(pairs.size, pairs))
    assert g.m > 1_000_000
    print(f"[case] few slices n={g.n} m={g.m}", flush=True)
    want = oracle.method_census(dense, 4)  # (the pairs have no connected set of four)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    assert np.array_equal(pm.census(off, idx, g.n, 4), want)
    h3, h4 = pm.census_multi(off, idx, g.n, (3, 4))
    assert np.array_equal(h4, want) and np.array_equal(h3, oracle.method_census(dense, 3))
