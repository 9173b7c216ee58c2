"""Workloads whose speed is watched: what users of the census library call,
from the smallest network to the largest, with the inputs each call starts
from.

listed() names the fixed ones, draw(rng) gives another of the same ranges.
A case is a dict of plain values; its "kind" selects the entry point:

  census      one graph, one size (out-CSR alone or with the in-CSR)
  multi       one graph, several sizes over one build (a motif profile)
  undirected  the undirected census of one graph
  batch       one fused census of an ensemble of graphs
  null        the whole null-model job: randomise, census, z-scores
  randomize   degree-preserving randomisation of an ensemble in place
  census6     motifs of size 6 of a small graph
  serve       a burst of host requests through the census server

Graphs are seeded Chung-Lu power-law digraphs (or uniform G(n, m)) with a
reciprocated fraction, the shape of the networks the benchmark and the tests
use; sizes are theirs too.
"""
import atexit
import itertools

import numpy as np
import torch

import paper_1203_3415_amd as pm

DEV = "cuda:0"
CLASSES = {3: 13, 4: 199, 5: 9364}


# ------------------------------------------------------------------ cases --

def listed():
    return [
        # the smallest call: one small network, counts wanted on the host
        {"name": "tiny_k3", "kind": "census", "n": 160, "m": 520, "gout": 2.5, "gin": 2.5, "r": 0.1, "ks": "3",
         "in_csr": False, "shuffled": False, "host": True},
        # a motif profile of a network of about a thousand vertices
        {"name": "profile_small", "kind": "multi", "n": 1000, "m": 5500, "gout": 0.0, "gin": 0.0, "r": 0.18,
         "ks": "345", "in_csr": True, "shuffled": False, "host": False},
        # the benchmark's default step: k = 3 and 4 of a large network
        {"name": "profile_large", "kind": "multi", "n": 100000, "m": 1000000, "gout": 2.1, "gin": 2.1, "r": 0.2,
         "ks": "34", "in_csr": True, "shuffled": False, "host": False},
        # a large network straight from an arc list: rows unsorted, no in-CSR
        {"name": "k3_unsorted", "kind": "census", "n": 100000, "m": 1000000, "gout": 2.1, "gin": 2.1, "r": 0.2,
         "ks": "3", "in_csr": False, "shuffled": True, "host": False},
        # an ordinary network of odd sizes at k = 4
        {"name": "k4_ragged", "kind": "census", "n": 20011, "m": 100003, "gout": 2.3, "gin": 2.4, "r": 0.15,
         "ks": "4", "in_csr": False, "shuffled": False, "host": False},
        # the benchmark's k = 5 network
        {"name": "k5_large", "kind": "census", "n": 20000, "m": 100000, "gout": 2.2, "gin": 2.5, "r": 0.1,
         "ks": "5", "in_csr": True, "shuffled": False, "host": False},
        # an undirected network, each edge listed once
        {"name": "undirected_k4", "kind": "undirected", "n": 30011, "m": 150013, "gout": 2.3, "gin": 2.3, "r": 0.0,
         "ks": "4", "in_csr": False, "shuffled": False, "host": False},
        # one fused census of an ensemble of graphs of uneven sizes
        {"name": "ensemble_k4", "kind": "batch", "count": 501, "n": 500, "n_max": 5000, "per": 4, "gout": 2.3,
         "gin": 2.3, "r": 0.05, "ks": "4"},
        # the null-model job of the benchmark: 1,000 randomisations of one graph
        {"name": "null_job", "kind": "null", "n": 2000, "m": 8000, "count": 1000, "spa": 100, "gout": 2.3, "gin": 2.3,
         "r": 0.05, "ks": "4", "mutual": False},
        # an uneven ensemble randomised with reciprocated pairs kept
        {"name": "randomize_mutual", "kind": "randomize", "count": 256, "n": 500, "n_max": 5000, "per": 4,
         "spa": 100, "gout": 2.3, "gin": 2.3, "r": 0.1, "mutual": True},
        # motifs of size 6 of a small network
        {"name": "census6_small", "kind": "census6", "n": 300, "m": 700, "gout": 2.5, "gin": 2.5, "r": 0.1},
        # a burst of mixed requests from host buffers through the server
        {"name": "serve_burst", "kind": "serve", "requests": 24, "m_min": 1000, "m_max": 100000, "k5_max": 20000,
         "gout": 2.4, "gin": 2.4, "r": 0.1},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["census", "census", "multi", "undirected", "batch", "null", "randomize", "census6", "serve"])
    g = {"gout": round(rng.uniform(2.25, 2.6), 3), "gin": round(rng.uniform(2.25, 2.6), 3),
         "r": round(rng.uniform(0.0, 0.25), 3)}
    if kind in ("census", "multi", "undirected"):
        ks = rng.choice(["3", "4", "5"]) if kind != "multi" else rng.choice(["34", "45", "345"])
        m = _log_int(rng, 300, 25000 if "5" in ks else 600000)
        n = max(40, int(m / rng.uniform(3.0, 12.0)))
        c = {"kind": kind, "n": n, "m": m, "ks": ks, "in_csr": kind != "undirected" and rng.random() < 0.5,
             "shuffled": False, "host": rng.random() < 0.3, **g}
        c["shuffled"] = not c["in_csr"] and rng.random() < 0.5
        if kind == "undirected":
            c["r"] = 0.0
        if rng.random() < 0.2:
            c["gout"] = c["gin"] = 0.0  # uniform G(n, m)
        return c
    if kind == "batch":
        lo = _log_int(rng, 60, 2000)
        return {"kind": kind, "count": _log_int(rng, 8, 400), "n": lo, "n_max": int(lo * rng.uniform(1.0, 2.5)),
                "per": rng.choice([2, 3, 4, 5]), "ks": rng.choice(["3", "4", "4"]), **g}
    if kind == "null":
        n = _log_int(rng, 150, 2000)
        return {"kind": kind, "n": n, "m": int(n * rng.uniform(2.0, 4.0)), "count": _log_int(rng, 30, 800),
                "spa": rng.choice([20, 50, 100]), "ks": rng.choice(["3", "4"]), "mutual": rng.random() < 0.3, **g}
    if kind == "randomize":
        lo = _log_int(rng, 100, 2500)
        return {"kind": kind, "count": _log_int(rng, 8, 256), "n": lo, "n_max": int(lo * rng.uniform(1.0, 2.0)),
                "per": rng.choice([2, 3, 4]), "spa": rng.choice([20, 50, 100]), "mutual": rng.random() < 0.5, **g}
    if kind == "census6":
        m = _log_int(rng, 150, 700)
        return {"kind": kind, "n": max(60, int(m / rng.uniform(1.8, 2.6))), "m": m, **g}
    lo = _log_int(rng, 600, 5000)
    return {"kind": "serve", "requests": rng.randrange(8, 25), "m_min": lo, "m_max": int(lo * rng.uniform(2, 20)),
            "k5_max": 15000, **g}


# ----------------------------------------------------------------- graphs --

def _cdf(n, gamma, rng, permute):
    w = (np.arange(n, dtype=np.float64) + 1.0) ** (-1.0 / (gamma - 1.0)) if gamma else np.ones(n)
    if permute:
        w = w[rng.permutation(n)]
    c = np.cumsum(w)
    return c / c[-1]


def _arcs(n, m, gout, gin, r, rng):
    """m distinct arcs as sorted keys u * n + v, about a fraction r of them
    reciprocated; out-weights fall with the index, in-weights are permuted."""
    m = min(m, n * (n - 1) // 2)
    base = m - int(round(m * r / 2))
    co, ci = _cdf(n, gout, rng, False), _cdf(n, gin, rng, True)
    keys = np.zeros(0, np.int64)
    while keys.size < base:
        need = int((base - keys.size) * 1.3) + 64
        u = np.minimum(np.searchsorted(co, rng.random(need), side="right"), n - 1)
        v = np.minimum(np.searchsorted(ci, rng.random(need), side="right"), n - 1)
        k = u * np.int64(n) + v
        keys = np.unique(np.concatenate([keys, k[u != v]]))
    keys = keys[np.sort(rng.permutation(keys.size)[:base])]
    rev = (keys % n) * n + keys // n
    cand = rev[~np.isin(rev, keys, assume_unique=True)]
    add = cand[rng.permutation(cand.size)[:m - base]]
    return np.sort(np.concatenate([keys, add]))


def _once(keys, n):
    """Each unordered pair kept once (as the arc listed first)."""
    u, v = keys // n, keys % n
    _, first = np.unique(np.minimum(u, v) * n + np.maximum(u, v), return_index=True)
    return keys[np.sort(first)]


def _csr(keys, n):
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(keys // n, minlength=n), out=off[1:])
    return off.astype(np.int32), (keys % n).astype(np.int32)


def _graph(case, seed):
    rng = np.random.default_rng([seed, 101])
    n = case["n"]
    keys = _arcs(n, case["m"], case["gout"], case["gin"], case["r"], rng)
    if case["kind"] == "undirected":
        keys = _once(keys, n)
    off, idx = _csr(keys, n)
    ioff = iidx = None
    if case.get("in_csr"):
        ioff, iidx = _csr(np.sort((keys % n) * n + keys // n), n)
    if case.get("shuffled"):  # rows in the order of an arc list
        p = rng.permutation(keys.size)
        idx = idx[p[np.argsort(keys[p] // n, kind="stable")]]
    return off, idx, ioff, iidx


def _ensemble(case, seed):
    rng = np.random.default_rng([seed, 202])
    sizes = np.random.default_rng(202).integers(case["n"], case["n_max"] + 1, case["count"])  # the same for every seed
    out = []
    for n in sizes.tolist():
        out.append((n, *_csr(_arcs(n, case["per"] * n, case["gout"], case["gin"], case["r"], rng), n)))
    return out


def _on_device(graphs):
    """The ensemble's targets in one device buffer (rows of graph i at a
    16-byte boundary), its offsets in another; views per graph."""
    ooff, iooff, no, ni = [], [], 0, 0
    for n, off, idx in graphs:
        ooff.append(no)
        iooff.append(ni)
        no += (off.size + 3) // 4 * 4
        ni += (idx.size + 3) // 4 * 4
    flat_off, flat_idx = np.zeros(max(no, 1), np.int32), np.zeros(max(ni, 1), np.int32)
    for (n, off, idx), a, b in zip(graphs, ooff, iooff):
        flat_off[a:a + off.size] = off
        flat_idx[b:b + idx.size] = idx
    do, di = torch.from_numpy(flat_off).to(DEV), torch.from_numpy(flat_idx).to(DEV)
    views = [(do[a:a + off.size], di[b:b + idx.size], n) for (n, off, idx), a, b in zip(graphs, ooff, iooff)]
    return views, di


# ------------------------------------------------------------ prepare, run --

_SERVER = None


def _server():
    """One server for the process, as a serving program keeps it."""
    global _SERVER
    if _SERVER is None:
        _SERVER = pm.Server(6 << 30, max_inflight=4)
        atexit.register(_SERVER.close)
    return _SERVER


def _serve_sizes(case):
    q = case["requests"]
    out = []
    for i in range(q):
        m = int(round(case["m_min"] * (case["m_max"] / case["m_min"]) ** (i / max(1, q - 1))))
        k = (3, 4, 5)[i % 3]
        out.append((max(10, m // 5), m, 4 if k == 5 and m > case["k5_max"] else k))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("census", "multi", "undirected", "census6", "null"):
        off, idx, ioff, iidx = _graph(case, seed)
        st = {"case": case, "n": case["n"]}
        st["off"], st["idx"] = pm.to_device(off, idx, DEV)
        st["ioff"], st["iidx"] = pm.to_device(ioff, iidx, DEV) if ioff is not None else (None, None)
        if kind == "census6":
            st["out"] = torch.empty(pm.NUM_CLASSES6, dtype=torch.int64, device=DEV)
        elif kind == "null":
            C = CLASSES[int(case["ks"])]
            st["seed"] = seed
            st["out"] = torch.empty((case["count"] + 1, C), dtype=torch.int64, device=DEV)
            st["z"] = torch.empty(C, dtype=torch.float64, device=DEV)
        elif kind == "undirected":
            st["out"] = torch.empty({3: 2, 4: 6, 5: 21}[int(case["ks"])], dtype=torch.int64, device=DEV)
        else:
            st["outs"] = [torch.empty(CLASSES[int(k)], dtype=torch.int64, device=DEV) for k in case["ks"]]
        return st
    if kind in ("batch", "randomize"):
        graphs, flat = _on_device(_ensemble(case, seed))
        st = {"case": case, "graphs": graphs, "seed": seed}
        if kind == "batch":
            st["out"] = torch.empty((len(graphs), CLASSES[int(case["ks"])]), dtype=torch.int64, device=DEV)
        else:
            st["flat"], st["fresh"] = flat, flat.clone()
        return st
    rng = np.random.default_rng([seed, 303])
    reqs = []
    for n, m, k in _serve_sizes(case):
        off, idx = _csr(_arcs(n, m, case["gout"], case["gin"], case["r"], rng), n)
        reqs.append((off, idx, n, k))
    return {"case": case, "requests": reqs, "server": _server()}


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "census":
        out = None if c["host"] else state["outs"][0]
        return pm.census(state["off"], state["idx"], state["n"], int(c["ks"]), in_off=state["ioff"],
                         in_idx=state["iidx"], out=out)
    if kind == "multi":
        return pm.census_multi(state["off"], state["idx"], state["n"], [int(k) for k in c["ks"]],
                               in_off=state["ioff"], in_idx=state["iidx"], outs=None if c["host"] else state["outs"])
    if kind == "undirected":
        return pm.census_undirected(state["off"], state["idx"], state["n"], int(c["ks"]),
                                    out=None if c["host"] else state["out"])
    if kind == "batch":
        return pm.census_batch(state["graphs"], int(c["ks"]), out=state["out"])
    if kind == "null":
        return pm.null_model(state["off"], state["idx"], state["n"], c["count"], int(c["ks"]), c["spa"],
                             state["seed"], out=state["out"], z_out=state["z"], mutual=c["mutual"])
    if kind == "randomize":
        state["flat"].copy_(state["fresh"])  # the same ensemble again
        pm.null_randomize(state["graphs"], c["spa"], state["seed"], mutual=c["mutual"])
        return state["flat"]
    if kind == "census6":
        return pm.census6(state["off"], state["idx"], state["n"], out=state["out"])
    srv = state["server"]
    tickets = [srv.submit(off, idx, n, k) for off, idx, n, k in state["requests"]]
    return [srv.wait(t) for t in tickets]


# ------------------------------------------------------------- work, exact --

def work(case):
    """Bytes: each input read once, each output written once.  flops: the
    attempted arc switches of the randomising calls (their number is part of
    the request); the census has no operation count of its own."""
    kind = case["kind"]
    if kind in ("census", "multi", "undirected", "census6"):
        sides = 2 if case.get("in_csr") else 1
        inp = sides * 4 * (case["n"] + 1 + case["m"])
        if kind == "census6":
            out = 8 * 1530843
        elif kind == "undirected":
            out = 8 * {3: 2, 4: 6, 5: 21}[int(case["ks"])]
        else:
            out = 8 * sum(CLASSES[int(k)] for k in case["ks"])
        return {"bytes": inp + out, "flops": 0}
    if kind == "null":
        C = CLASSES[int(case["ks"])]
        return {"bytes": 4 * (case["n"] + 1 + case["m"]) + 8 * C * (case["count"] + 2),
                "flops": case["count"] * case["spa"] * case["m"]}
    if kind in ("batch", "randomize"):
        n = case["count"] * (case["n"] + case["n_max"]) / 2
        m = n * case["per"]
        if kind == "batch":
            return {"bytes": 4 * (n + m) + 8 * CLASSES[int(case["ks"])] * case["count"], "flops": 0}
        return {"bytes": 4 * (n + 2 * m), "flops": m * case["spa"]}
    return {"bytes": sum(4 * (n + 1 + m) + 8 * CLASSES[k] for n, m, k in _serve_sizes(case)), "flops": 0}


def _triads(off, idx, n):
    """The k = 3 census by the definition: every vertex triple, its 6-bit
    code, the least code over the six orders, connected codes ranked."""
    bit = lambda i, j: i * 2 + (j if j < i else j - 1)  # noqa: E731
    canon = np.zeros(64, np.int64)
    conn = np.zeros(64, bool)
    for code in range(64):
        arcs = [(i, j) for i in range(3) for j in range(3) if i != j and code >> bit(i, j) & 1]
        canon[code] = min(sum(1 << bit(p[i], p[j]) for i, j in arcs) for p in itertools.permutations(range(3)))
        conn[code] = len({frozenset(a) for a in arcs}) >= 2
    ids = {c: i for i, c in enumerate(sorted({int(canon[c]) for c in range(64) if conn[c]}))}
    a = np.zeros((n, n), np.int64)
    a[np.repeat(np.arange(n), np.diff(off)), idx] = 1
    cnt = np.zeros(64, np.int64)
    up = np.triu(np.ones((n, n), bool), 1)
    for x in range(n - 2):
        s = slice(x + 1, n)
        sub, o, i = a[s, s], a[x, s], a[s, x]
        code = ((o[:, None] << bit(0, 1)) | (o[None, :] << bit(0, 2)) | (i[:, None] << bit(1, 0))
                | (i[None, :] << bit(2, 0)) | (sub << bit(1, 2)) | (sub.T << bit(2, 1)))
        cnt += np.bincount(code[up[s, s]], minlength=64)
    out = np.zeros(13, np.uint64)
    for code in range(64):
        if conn[code]:
            out[ids[int(canon[code])]] += np.uint64(cnt[code])
    return out


def exact(case, seed):
    """The triad census of a small graph by its definition; the larger counts
    would take minutes to hours that way."""
    if case["kind"] != "census" or case["ks"] != "3" or case["n"] > 600:
        return None
    off, idx, _, _ = _graph(case, seed)
    h = _triads(off, idx, case["n"])
    return h if case["host"] else h.view(np.int64)
