"""Arc-switch rounds against the host rendering of the chain, target by target, on
every instance of the switch kernel: two workgroups per CU (more graphs than CUs),
one per CU with and without the second set of reservations, and global memory;
for graphs with a few long rows (scanned by the wave), with many rows of middling
length (scanned by their lanes) and with rows on both sides of where the scans
change hands."""
import numpy as np
import pytest

import graphgen as gg
from test_gpu_switch_rounds import _graph, _switch

pytestmark = pytest.mark.gpu

SHAPES = {
    "hubs": (200, [1, 15, 16, 17, 18, 63, 64, 65, 127, 128, 129, 180]),
    "middling": (110, [17 + (7 * i) % 15 for i in range(110)]),
    "edges": (160, [w for w in (1, 7, 8, 9, 14, 15, 16, 17, 18, 62, 63, 64, 65, 66, 67) for _ in range(9)]),
}


@pytest.mark.parametrize("mutual", [False, True])
@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("place", ["two_per_cu", "one_per_cu", "one_set", "global"])
def test_paths_equal_host(place, shape, mutual):
    import torch
    import paper_1203_3415_amd as pm
    n, lens = SHAPES[shape]
    g = _graph(n, lens, 0.3, len(lens))
    if place in ("one_set", "global"):  # among isolated vertices: no room for a second set of n words, or for any
        n = {"one_set": 12000 if mutual else 15000, "global": 40000}[place]
        g = gg.from_arcs(n, g.arcs())
    lds, half = 38 * 1024, (g.m + 1) // 2
    words = n + 1 + half + (2 if mutual else 1) * n
    if place == "one_set":
        assert words <= lds < words + half + n
    assert (words > lds) == (place == "global")
    count = torch.cuda.get_device_properties(0).multi_processor_count + 40 if place == "two_per_cu" else 2
    off, idx = pm.to_device(g.out_off, g.out_idx)
    devs = [(off, idx.clone(), n) for _ in range(count)]
    print(f"[case] switch paths {place} {shape} mutual={mutual} m={g.m} graphs={count}", flush=True)
    pm.null_randomize(devs, 5, seed=11, mutual=mutual)
    torch.cuda.synchronize()
    for i in {0, 1, count // 2, count - 1}:
        assert devs[i][1].cpu().tolist() == _switch(g, 5, 11, i, mutual), i


def test_uneven_ensemble_is_checked():
    # 1,500 small graphs and a large one whose last target is wrong
    import torch
    import paper_1203_3415_amd as pm
    small = pm.to_device(np.array([0, 2, 3, 4], np.int32), np.array([1, 2, 0, 1], np.int32))
    n = 300000
    off = np.arange(n + 1, dtype=np.int32)
    idx = ((np.arange(n) + 1) % n).astype(np.int32)
    for last, name in ((n, "EINDEX"), (n - 1, "ESELFLOOP"), (0, None)):
        idx[-1] = last
        o, x = pm.to_device(off, idx)
        devs = [(small[0], small[1].clone(), 3) for _ in range(1500)] + [(o, x, n)]
        print(f"[case] uneven ensemble, last target {last}", flush=True)
        if name is None:
            pm.null_randomize(devs, 1, seed=1)
            torch.cuda.synchronize()
            assert np.array_equal(np.sort(x.cpu().numpy()), np.arange(n))
        else:
            with pytest.raises(pm.MotifError) as e:
                pm.null_randomize(devs, 1, seed=1)
            assert e.value.name == name and np.array_equal(x.cpu().numpy(), idx)


@pytest.mark.parametrize("seed", range(4))
def test_repeated_arcs_alike_in_lds_and_memory(seed):
    # repeated arcs are not refused; the reverse of one may then be gone from its row
    import torch
    import paper_1203_3415_amd as pm
    rng = np.random.default_rng(seed)
    pairs = [(int(a), int(b)) for a, b in rng.integers(0, 30, (150, 2)) if a != b]
    arcs = sorted(pairs + [(b, a) for a, b in pairs[::2]] + pairs[::3])
    off = np.searchsorted([a for a, _ in arcs], np.arange(31)).astype(np.int32)
    idx = np.asarray([b for _, b in arcs], np.int32)
    far = np.concatenate([off, np.full(40000 - 30, len(arcs), np.int32)])
    o, x = pm.to_device(off, idx)
    fo, fx = pm.to_device(far, idx)
    print(f"[case] repeated arcs seed={seed} m={len(arcs)}", flush=True)
    pm.null_randomize([(o, x, 30)], 40, seed=seed, mutual=True)
    pm.null_randomize([(fo, fx, 40000)], 40, seed=seed, mutual=True)
    torch.cuda.synchronize()
    assert torch.equal(x, fx)
