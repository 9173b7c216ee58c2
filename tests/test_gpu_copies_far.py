"""GPU tests of the k = 4 census on graphs of many ids (more than 32 blocks of
12,288), where vertices of some thousand visits have their wedges hashed in parts:
both widths of the counts, their edges (127 and 1,024 lower neighbours, 3,072 and
65,536 visits), a part that holds more vertices than its hash and is halved, and
a batch.  Counts are whole numbers and compared exactly with the per-anchor method
on the CPU."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_copies import check, from_edges

pytestmark = pytest.mark.gpu
N = 400000


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


def _pole(mids, each, ends, rng, high=0, n=N):
    """A pole over `mids` vertices of `each` further neighbours among `ends`, with `high` leaves of its own (lower
    neighbours too) or, with high < 0, -high neighbours of higher degree."""
    at = [1]

    def fresh(k):
        at[0] += k
        return np.arange(at[0] - k, at[0])
    m = fresh(mids)
    e = [np.c_[np.zeros(mids, np.int64), m],
         np.c_[np.repeat(m, each), np.concatenate([rng.choice(ends, each, replace=False) for _ in range(mids)])]]
    if high > 0:
        e.append(np.c_[np.zeros(high, np.int64), fresh(high)])
    if high < 0:
        top = fresh(-high)
        own = mids - high + 50  # leaves of each: more than the pole's neighbours
        e += [np.c_[np.zeros(-high, np.int64), top], np.c_[np.repeat(top, own), fresh(-high * own)]]
    assert at[0] <= n // 2
    return np.concatenate(e)


@pytest.mark.parametrize("mids,each,high", [(127, 40, -60), (128, 40, 60), (100, 30, -40), (100, 29, -40), (1024, 20, 0),
                                            (1025, 20, 0), (600, 108, 0), (600, 109, 0), (127, 40, 0),
                                            (128, 40, 0)])
def test_pole(pm, mids, each, high):
    # far ends: 3,000 vertices spread over the ids, so that many are met twice
    rng = np.random.default_rng(mids * each)
    ends = N // 2 + rng.choice(N // 2, 3000, replace=False)
    check(pm, from_edges(N, *_pole(mids, each, ends, rng, high).T, rng, shuffle=False), 4, "pole")


@pytest.mark.parametrize("mids,high", [(110, -320), (150, 600)])
def test_crowded_part(pm, mids, high):
    # far ends whose mixed ids share their low bits: one part holds them all
    n = 1 << 20
    h = np.arange(n, dtype=np.uint64)
    m32 = np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(16)
    h = h * np.uint64(0x85EBCA6B) & m32
    h ^= h >> np.uint64(13)
    h = h * np.uint64(0xC2B2AE35) & m32
    h ^= h >> np.uint64(16)
    ends = np.flatnonzero(h % np.uint64(64) == 5)
    ends = ends[ends >= n // 2]
    assert len(ends) > 8000
    rng = np.random.default_rng(high + 1000)
    check(pm, from_edges(n, *_pole(mids, 400, ends, rng, high, n).T, rng, shuffle=False), 4, "crowded part")


def test_power_law_and_batch(pm):
    g = gg.chung_lu(500000, 600000, 2.1, 2.2, 0.1, seed=8)
    check(pm, g, 4, "power law")
    rng = np.random.default_rng(1)
    ends = N // 2 + rng.choice(N // 2, 3000, replace=False)
    p = from_edges(N, *_pole(200, 50, ends, rng, 0).T, rng)
    print("[case] batch with many ids", flush=True)
    h = pm.census_batch([(*pm.to_device(x.out_off, x.out_idx), x.n) for x in (g, p, g)], 4)
    want = oracle.method_census(g, 4)
    assert np.array_equal(h[0], want) and np.array_equal(h[2], want)
    assert np.array_equal(h[1], oracle.method_census(p, 4))
