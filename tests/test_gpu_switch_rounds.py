"""Arc-switch rounds against a plain host rendering of the same chain, target
by target: rows on both sides of the lengths at which the row scans change
hands (one lane, the whole wave, several steps of it), in LDS and in global
memory, for both kinds of switch."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu
M64 = (1 << 64) - 1
GAMMA = 0x9E3779B97F4A7C15


def _mix(z):
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & M64
    return z ^ (z >> 31)


def _switch(g, per_arc, seed, graph, mutual):
    """The chain of one graph: rounds of 1,024 proposals; a row goes to its
    lowest proposal; a proposal with both rows switches when that is valid."""
    off = g.out_off.astype(int).tolist()
    idx = g.out_idx.astype(int).tolist()
    m = len(idx)
    row = np.repeat(np.arange(g.n), np.diff(g.out_off)).tolist()
    have = [set(idx[off[v]:off[v + 1]]) for v in range(g.n)]
    kind = [row[s] in have[idx[s]] for s in range(m)]
    perm = [s for s in range(m) if kind[s]] + [s for s in range(m) if not kind[s]]
    nmut = sum(kind)
    key = _mix((seed + (graph + 1) * GAMMA) & M64)
    for r in range((per_arc * m + 1023) // 1024):
        lock, props = {}, []
        for t in range(1024):
            x = _mix((key + (r * 1024 + t + 1) * GAMMA) & M64)
            i = ((x & 0xFFFFFFFF) * m) >> 32
            j = ((x >> 32) * m) >> 32
            if mutual:
                lo, nk = (0, nmut) if i < nmut else (nmut, m - nmut)
                j, i = perm[lo + (((x >> 32) * nk) >> 32)], perm[i]
            a, c = row[i], row[j]
            props.append((t, i, j, a, c))
            if a != c:
                lock.setdefault(a, t)
                lock.setdefault(c, t)
        won = [p for p in props if p[3] != p[4] and lock[p[3]] == p[0] and lock[p[4]] == p[0]]
        run = won
        if mutual:
            held = {v: p[0] for p in won for v in p[3:5]}
            claim = {}
            for t, i, j, a, c in won:
                claim.setdefault(idx[i], t)
                claim.setdefault(idx[j], t)
            run = [p for p in won if all(claim[v] == p[0] and held.get(v, p[0]) == p[0] for v in (idx[p[1]], idx[p[2]]))]
        for t, i, j, a, c in run:
            b, d = idx[i], idx[j]
            if a == d or c == b or b == d or d in have[a] or b in have[c]:
                continue
            if mutual and (a in have[d] or c in have[b]):
                continue
            idx[i], idx[j] = d, b
            have[a] = have[a] - {b} | {d}
            have[c] = have[c] - {d} | {b}
            if mutual and kind[i]:
                s = off[b] + idx[off[b]:off[b + 1]].index(a)
                q = off[d] + idx[off[d]:off[d + 1]].index(c)
                idx[s], idx[q] = c, a
                have[b] = have[b] - {a} | {c}
                have[d] = have[d] - {c} | {a}
    return idx


def _graph(n, lens, recip, seed):
    """Rows of the given lengths first, short ones after; some arcs answered."""
    rng = np.random.default_rng(seed)
    arcs = set()
    for v in range(n):
        for w in rng.permutation(n - 1)[:lens[v] if v < len(lens) else int(rng.integers(0, 4))]:
            arcs.add((v, int(w) + (int(w) >= v)))
    for u, v in sorted(arcs):
        if v >= len(lens) and rng.random() < recip:
            arcs.add((v, u))
    return gg.from_arcs(n, sorted(arcs))


LENS = [1, 15, 16, 17, 18, 63, 64, 65, 127, 128, 129, 180]


@pytest.mark.parametrize("mutual", [False, True])
@pytest.mark.parametrize("place", ["half_lds", "full_lds", "global"])
def test_switch_rounds_equal_host(place, mutual):
    import torch
    import paper_1203_3415_amd as pm
    g = _graph(200, LENS, 0.3, 9)
    if place != "half_lds":  # the same graph among isolated vertices: more offsets and locks
        g = gg.from_arcs({"full_lds": 11000, "global": 40000}[place], g.arcs())
    off, idx = pm.to_device(g.out_off, g.out_idx)
    devs = [(off, idx.clone(), g.n) for _ in range(2)]
    print(f"[case] switch rounds {place} mutual={mutual} m={g.m}", flush=True)
    pm.null_randomize(devs, 12, seed=5, mutual=mutual)
    torch.cuda.synchronize()
    for i in range(2):
        assert devs[i][1].cpu().tolist() == _switch(g, 12, 5, i, mutual)
