"""GPU tests of the outcome of calls whose input is found wrong while other work
of the call is on the device."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_3415_amd as pm
    pm.lib()
    return pm


def _hubs(n, hubs, leaves, seed):
    """A power-law graph whose first vertices are joined to many of the rest."""
    rng = np.random.default_rng(seed)
    base = gg.chung_lu(n, 4 * n, 2.2, 2.3, 0.2, seed=seed).arcs()
    extra = [(h, int(w)) for h in range(hubs) for w in rng.choice(np.arange(hubs, n), leaves, replace=False)]
    return gg.from_arcs(n, np.unique(np.concatenate([base, np.asarray(extra, np.int64)]), axis=0))


# k = 5 of a graph of more than 65,536 vertices takes the core-reuse kernel,
# beside which the check runs
@pytest.mark.parametrize("n,ks,schemes", [(5000, (3, 4), (1, 2)), (5000, (4,), (1, 2)), (70000, (3, 4, 5), (1,))])
def test_in_csr_checked_beside_the_censuses(pm, n, ks, schemes):
    import torch
    g = _hubs(n, 8, 1500, seed=n)
    rng = np.random.default_rng(n)
    in_off, in_idx = g.in_csr()
    for v in range(n):  # rows out of order: the placement of sorted rows is not taken
        a, b = int(in_off[v]), int(in_off[v + 1])
        in_idx[a:b] = rng.permutation(in_idx[a:b])
    wrong = in_idx.copy()
    v = int(np.argmax(np.diff(in_off)))
    listed = set(in_idx[in_off[v]:in_off[v + 1]].tolist())
    wrong[in_off[v]] = next(w for w in range(n - 1, -1, -1) if w != v and w not in listed)
    off, idx = pm.to_device(g.out_off, g.out_idx)
    saved = pm.get_tuning(4)
    try:
        for scheme in schemes:
            pm.set_tuning(4, heavy=scheme)
            want = [pm.census(off, idx, n, k) for k in ks]
            outs = [torch.empty(len(w), dtype=torch.int64, device=off.device) for w in want]
            for rep in range(4):
                print(f"[case] in-CSR beside n={n} ks={ks} scheme={scheme} round {rep}", flush=True)
                for o in outs:
                    o.fill_(-7)
                io, ii = pm.to_device(in_off, wrong)
                with pytest.raises(pm.MotifError) as e:
                    pm.census_multi(off, idx, n, ks, io, ii, outs=outs)
                assert e.value.name == "ETRANSPOSE"
                assert all((o == -7).all().item() for o in outs)
                io, ii = pm.to_device(in_off, in_idx)
                for got, w in zip(pm.census_multi(off, idx, n, ks, io, ii), want):
                    assert np.array_equal(got, w)
    finally:
        pm.set_tuning(4, **saved)


@pytest.mark.parametrize("bad,name", [(10 ** 6, "EINDEX"), (-1, "EINDEX"), ("self", "ESELFLOOP")])
def test_wrong_arc_is_named(pm, bad, name):
    # one wrong arc, met while most workgroups of the check are still to start
    g = gg.chung_lu(100000, 1000000, 2.1, 2.1, 0.2, seed=3)
    rng = np.random.default_rng(5)
    idx = g.out_idx.copy()
    for v in np.flatnonzero(np.diff(g.out_off) > 200):
        idx[g.out_off[v]:g.out_off[v + 1]] = rng.permutation(idx[g.out_off[v]:g.out_off[v + 1]])
    for place in (0, 5000, g.m - 1):
        wrong = idx.copy()
        wrong[place] = int(np.searchsorted(g.out_off, place, side="right")) - 1 if bad == "self" else bad
        off_t, idx_t = pm.to_device(g.out_off, wrong)
        for rep in range(8):
            print(f"[case] wrong arc {bad} at {place} round {rep}", flush=True)
            with pytest.raises(pm.MotifError) as e:
                pm.census(off_t, idx_t, g.n, 3)
            assert e.value.name == name
