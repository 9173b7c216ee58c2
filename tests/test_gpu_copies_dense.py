"""GPU tests of the k = 3, 4 censuses by subgraph copies where neighbourhoods are
dense: vertices of small dense graphs that get a workgroup each (41 higher
neighbours or more), the same cliques in graphs that keep the tiers by degree,
and neighbourhoods of more than 256 whose edges are few or many (K4s one by one
or by intersections, a lane per neighbour or per word).  Counts are whole numbers
and compared exactly with the per-anchor method on the CPU."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_copies import check, from_edges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


def _random(n, p, rng, r=0.4):
    a, b = np.triu_indices(n, 1)
    keep = rng.random(len(a)) < p
    return a[keep], b[keep], r


@pytest.mark.parametrize("p", [0.35, 0.6, 0.9, 1.0])
@pytest.mark.parametrize("n", [73, 104, 130, 180])
def test_dense_small(pm, n, p):
    rng = np.random.default_rng(n * 10 + int(10 * p))
    a, b, r = _random(n, p, rng)
    check(pm, from_edges(n, a, b, rng, r=r), 4, f"dense p={p}")


@pytest.mark.parametrize("n", [41, 42, 43, 65, 66, 129, 130])
def test_clique_among_many(pm, n):
    # a clique in a graph of 2,000 vertices: waves of one, two and more per vertex
    rng = np.random.default_rng(n)
    a, b, r = _random(n, 1.0, rng)
    c = np.arange(n, 2000)
    check(pm, from_edges(2000, np.concatenate([a, c]), np.concatenate([b, rng.integers(0, n, len(c))]), rng, r=r), 4,
          "clique among many")


@pytest.mark.parametrize("k", [3, 4])
@pytest.mark.parametrize("p", [0.02, 0.1, 0.9])
def test_wide_neighbourhood(pm, p, k):
    # eight vertices joined to 262 of higher degree, which a third set raises
    rng = np.random.default_rng(int(100 * p))
    nz = int(262 * (1.05 - p))
    x, y, z = np.arange(8), 8 + np.arange(262), 270 + np.arange(nz)
    a, b, r = _random(262, p, rng)
    e = np.concatenate([np.stack(np.meshgrid(x, y, indexing="ij"), -1).reshape(-1, 2),
                        np.stack(np.meshgrid(y, z, indexing="ij"), -1).reshape(-1, 2), np.c_[a + 8, b + 8]])
    check(pm, from_edges(270 + nz, e[:, 0], e[:, 1], rng, r=r), k, f"wide neighbourhood p={p}")
