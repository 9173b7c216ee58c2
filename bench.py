#!/usr/bin/env python3
"""Throughput benchmark of the MI355X motif census (one JSON line on stdout).

Default workload: Motifs-3 and Motifs-4 on a directed Chung-Lu power-law
digraph with n = 100,000 vertices and m = 1,000,000 arcs (in/out weight
exponent 2.1, reciprocity 0.2, seed 2).  One step = the exact census for k = 3
and for k = 4 of that graph, whose CSR is resident in HBM before timing starts
(validation, one typed-G* build shared by both sizes, the census kernels and
the exact divisions all run inside the step).  value = arcs censused per
second = m / (step time).

Other workloads (--workload): gnm_n1000 (k = 3,4,5 on a G(n,m) digraph with
n = 1000, m = 5000 + 10 % reciprocated), chunglu_n2e4_k5 (Motifs-5 on a
Chung-Lu digraph n = 20,000, m = 100,000, exponents 2.2/2.5, reciprocity 0.1),
nullmodel_k4 (batched null model: graphs per second, fused vs per-graph loop)
and serving (Poisson request stream: p50/p99 latency and throughput).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0


def _threads() -> int:
    try:
        return int(os.environ.get("OMP_NUM_THREADS") or os.cpu_count() or 1)
    except ValueError:
        return os.cpu_count() or 1


# ------------------------------------------------------------- workloads ---

def make_graph(name: str):
    import graphgen as gg
    if name == "chunglu_n1e5_k34":
        return gg.chung_lu(100_000, 1_000_000, 2.1, 2.1, 0.2, seed=2), (3, 4)
    if name in ("chunglu_n1e5_k3", "chunglu_n1e5_k4"):  # one size alone, for kernel timing
        return gg.chung_lu(100_000, 1_000_000, 2.1, 2.1, 0.2, seed=2), (int(name[-1]),)
    if name == "gnm_n1000":
        return gg.gnm_reciprocal(1000, 5000, 0.1, seed=1), (3, 4, 5)
    if name == "chunglu_n2e4_k5":
        return gg.chung_lu(20_000, 100_000, 2.2, 2.5, 0.1, seed=4), (5,)
    raise SystemExit(f"unknown workload {name}")


def graph_stats(g):
    """Degree-ordered structure of G* used for the algorithmic-byte counts:
    d*(v), d+(v), sum over neighbours of d+ (S+), per-vertex triangle counts."""
    n = g.n
    a = g.arcs()
    lo = np.minimum(a[:, 0], a[:, 1])
    hi = np.maximum(a[:, 0], a[:, 1])
    key = np.unique(lo * n + hi)
    u, v = key // n, key % n
    deg = np.bincount(u, minlength=n) + np.bincount(v, minlength=n)
    rank_u = deg[u] * n + u
    rank_v = deg[v] * n + v
    src = np.where(rank_u < rank_v, u, v)
    dst = np.where(rank_u < rank_v, v, u)
    order = np.lexsort((dst, src))
    src, dst = src[order], dst[order]
    dplus = np.bincount(src, minlength=n)
    poff = np.zeros(n + 1, np.int64)
    np.cumsum(dplus, out=poff[1:])
    # S+(v) = sum of d+ over all neighbours of v
    splus = np.bincount(u, weights=dplus[v], minlength=n) + np.bincount(v, weights=dplus[u], minlength=n)
    # triangles per vertex by oriented intersection
    tri = np.zeros(n, np.int64)
    mark = np.zeros(n, bool)
    for x in np.flatnonzero(dplus >= 2):
        nx = dst[poff[x]:poff[x + 1]]
        mark[nx] = True
        for w in nx:
            cand = dst[poff[w]:poff[w + 1]]
            hit = cand[mark[cand]]
            if hit.size:
                tri[x] += hit.size
                tri[w] += hit.size
                np.add.at(tri, hit, 1)
        mark[nx] = False
    return dict(n=n, mstar=int(key.size), deg=deg, dplus=dplus, splus=splus, tri=tri, u=u, v=v)


def k4_kernel_bytes(st) -> float:
    """Algorithmic bytes of one k = 4 census kernel launch: per undirected
    edge e = {u,v} the two typed rows (4 (d_u + d_v) B) and, per vertex x of
    adj(e), its oriented row (4 d+(x) B) plus its two offsets (8 B).
    |adj(e)| = d_u + d_v - 2 - |N(u) ∩ N(v)|, summed with the triangle counts."""
    deg, dplus, splus, tri, u, v = st["deg"], st["dplus"], st["splus"], st["tri"], st["u"], st["v"]
    rows = 4.0 * float((deg.astype(np.float64) ** 2).sum())
    members = float((deg[u] + deg[v] - 2).sum()) - 3.0 * float(tri.sum() / 3)
    probes = float((splus[u] + splus[v]).sum() - (dplus[u] + dplus[v]).sum()) - float((dplus * tri).sum())
    return rows + 4.0 * probes + 8.0 * members


def _core_side(st):
    """Per undirected edge: the core (higher rank (d*, id)) and the side."""
    deg, u, v, n = st["deg"], st["u"], st["v"], st["n"]
    ru = deg[u].astype(np.int64) * n + u
    rv = deg[v].astype(np.int64) * n + v
    return np.where(ru > rv, u, v), np.where(ru > rv, v, u)


def kr4_kernel_bytes(st) -> float:
    """Algorithmic bytes of one launch of the k = 4 core-reuse kernel.
    Per core c (once): its typed row (4 d_c), the offsets (8 B) and N+ row
    (4 d+(y)) of every y in N(c), and one 4-byte W update per N+ entry:
    12 d_c + 8 S+(c).  Per anchor {c, s}: the side's row (4 d_s) and, for
    each of the d_s members q of R' = {s} u N(s) \ {c}, its offsets and W
    row (44 B) and its N+ row (4 d+(q)): 48 d_s + 4 (S+(s) - d+(c) + d+(s))."""
    deg = st["deg"].astype(np.float64)
    dplus = st["dplus"].astype(np.float64)
    splus = st["splus"]
    c, s = _core_side(st)
    anchor = 48.0 * deg[s] + 4.0 * (splus[s] - dplus[c] + dplus[s])
    cores = np.unique(c)
    return float(anchor.sum()) + float((12.0 * deg[cores] + 8.0 * splus[cores]).sum())


def kr5_kernel_bytes(st) -> float:
    """Algorithmic bytes of one launch of the k = 5 core-reuse kernel.  Per
    centre c (once): 12 d_c + 8 S+(c) as for k = 4.  Per connected triple
    (x, c, c2): the two side rows, 4 (d_x + d_c2), and per member q of
    N(x) u N(c2) its offsets and W row (44 B) and N+ row (4 d+(q)); the
    union is the sum over both rows minus the common neighbours, counted
    through the co-degrees t(c, q): sum over c != q of C(t, 2) g(q).
    Light triples (lighter side of degree <= 512) read the heavier side's
    part f(x) = 4 d_x + sum g(q) once per sub-chunk of at most 32 partners
    (and 768 table keys) instead of once per triple; the sub-chunks of a
    unit are counted as ceil(max(n_l / 32, sum(d + 1) / 768))."""
    import scipy.sparse as sp
    n, u, v = st["n"], st["u"], st["v"]
    deg = st["deg"].astype(np.float64)
    dplus = st["dplus"].astype(np.float64)
    A = sp.csr_matrix((np.ones(2 * len(u)), (np.r_[u, v], np.r_[v, u])), shape=(n, n))
    gq = 44.0 + 4.0 * dplus
    f = 4.0 * deg + A @ gq
    pairs = float(((deg - 1.0) * (A @ f)).sum())
    A2 = (A @ A).tocoo()
    off = A2.row != A2.col
    t = A2.data[off]
    inter = float((t * (t - 1.0) / 2.0 * gq[A2.col[off]]).sum())
    core = float((12.0 * deg + 8.0 * st["splus"])[deg >= 2].sum())
    # units (c, x): light partners are the neighbours of c of lower rank
    src, dst = np.r_[u, v], np.r_[v, u]
    key = deg * n + np.arange(n)  # rank (d*, id)
    order = np.lexsort((key[dst], src))
    cs, xs = src[order], dst[order]
    light = (deg[xs] <= 512).astype(np.float64)
    cl = np.cumsum(light) - light  # light entries before each position
    cd = np.cumsum(light * (deg[xs] + 1.0)) - light * (deg[xs] + 1.0)
    start = np.searchsorted(cs, cs, side="left")
    nl = cl - cl[start]
    sd = cd - cd[start]
    nsub = np.where(nl > 0, np.ceil(np.maximum(nl / 32.0, sd / 768.0)), 0.0)
    shared = float(((nl - nsub) * f[xs]).sum())
    return pairs - inter + core - shared


def k5_method_bytes(st) -> float:
    """The per-anchor byte model for k = 5 (what the paper's method, one
    connected triple at a time, reads): per triple (a, b, c) its three rows and the
    N+ rows of adj(T): 4 (d_a + d_b + d_c) + 4 sum over x in N(a), N(b), N(c)
    of d+(x).  Neighbourhood overlaps are not subtracted, so this is an upper
    estimate; triples are counted at their centre (a triangle three times)."""
    import scipy.sparse as sp
    n, u, v = st["n"], st["u"], st["v"]
    deg = st["deg"].astype(np.float64)
    A = sp.csr_matrix((np.ones(2 * len(u)), (np.r_[u, v], np.r_[v, u])), shape=(n, n))
    f = 4.0 * deg + 4.0 * st["splus"]
    pairs = deg * (deg - 1.0) / 2.0
    return float((pairs * f + (deg - 1.0) * (A @ f)).sum())


def k3_kernel_bytes(st) -> float:
    """Algorithmic bytes of one k = 3 census kernel launch: every typed G*
    entry with its row index (8 B, type counts), and per vertex u its row
    N+(u) (4 d+(u)) plus, for each w in N+(u), the offsets and row N+(w)
    (8 + 4 d+(w)); w is reached from its d*(w) - d+(w) lower-ranked
    neighbours."""
    deg, dplus = st["deg"].astype(np.float64), st["dplus"].astype(np.float64)
    return float(8.0 * deg.sum() + 4.0 * dplus.sum() + ((deg - dplus) * (8.0 + 4.0 * dplus)).sum())


def _lower_visits(st) -> float:
    """Entries of G* rows read for the wedges of every vertex's lower-ranked
    neighbours: the sum of d(v) over edges v -> u, v of lower rank."""
    _, side = _core_side(st)
    return float(st["deg"].astype(np.float64)[side].sum())


def copies4_bytes(st) -> float:
    """Algorithmic bytes of one k = 4 census by subgraph copies: the triangles
    as for k = 3, nine counters per edge written and read (72 B), the row
    entries of the wedges (4 B each) and the typed degrees of each edge's ends
    (32 B)."""
    return k3_kernel_bytes(st) + 104.0 * st["mstar"] + 4.0 * _lower_visits(st)


def copies5_bytes(st) -> float:
    """Algorithmic bytes of one k = 5 census by subgraph copies: the k = 4
    pass, the rows of all neighbours of every vertex (4 B per wedge end), the
    links of each triangle (six of 12 B, written and read) and the wedges of
    lower neighbours once more."""
    deg = st["deg"].astype(np.float64)
    return copies4_bytes(st) + 4.0 * float((deg ** 2).sum()) + 48.0 * float(st["tri"].sum()) + 4.0 * _lower_visits(st)


# ------------------------------------------------------------ main bench ---

def bench_census(args):
    import torch
    import paper_1203_3415_amd as pm

    g, ks = make_graph(args.workload)
    dev = torch.device("cuda:0")
    off, idx = pm.to_device(g.out_off, g.out_idx, dev)
    ioff, iidx = pm.to_device(*g.in_csr(), dev)
    outs = {k: torch.empty(pm.NUM_CLASSES[k], dtype=torch.int64, device=dev) for k in ks}
    torch.cuda.synchronize()

    def step():  # out- and in-CSR validated, one shared G* build for all sizes of the workload
        pm.census_multi(off, idx, g.n, ks, in_off=ioff, in_idx=iidx, outs=[outs[k] for k in ks])

    for _ in range(args.warmup):
        step()
    ref = {k: outs[k].cpu().numpy().view(np.uint64).copy() for k in ks}

    # in the timed steps, events bracket the census kernels only; the build
    # is timed in two more steps afterwards
    pm.profile_enable(True, census_only=True)
    kern_ms = {k: [] for k in ks}
    build_ms = {k: [] for k in ks}
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
        for k in ks:
            kern_ms[k].append(pm.profile_read(k)[0])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    pm.profile_enable(True)
    for _ in range(2):
        step()
        for k in ks:
            build_ms[k].append(pm.profile_read(k)[1])
    pm.profile_enable(False)
    ms_per_step = (t1 - t0) * 1000.0 / args.steps
    # the same histogram on every step (counts are exact integers)
    stable = all(np.array_equal(outs[k].cpu().numpy().view(np.uint64), ref[k]) for k in ks)

    st = graph_stats(g)
    checks = {"stable_across_steps": bool(stable)}
    if 3 in ks:
        wedges = int((st["deg"] * (st["deg"] - 1) // 2).sum())
        t_total = int(st["tri"].sum() // 3)
        checks["k3_sum_equals_wedges_minus_2T"] = int(ref[3].sum()) == wedges - 2 * t_total

    dominant = max(ks)
    kms = float(np.mean(kern_ms[dominant]))
    kname = kernel_name(dominant, pm.get_tuning(dominant)["heavy"] if dominant > 3 else 0, g.n, g.m, len(ks))
    kbytes = {"copies<3>": k3_kernel_bytes, "k4_kernel": k4_kernel_bytes, "copies<4>": copies4_bytes,
              "kr_kernel<4>": kr4_kernel_bytes, "copies<5>": copies5_bytes,
              "kr_kernel<5>": kr5_kernel_bytes}.get(kname, lambda _: None)(st)
    roofline = None
    if kbytes is not None:
        achieved = kbytes / (kms * 1e-3) / 1e9
        roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": stored_traffic(kname, args.workload),
                    "kernel": kname, "kernel_ms": round(kms, 3), "algorithmic_bytes": kbytes}
        # The per-anchor byte model (what the paper's method, one anchor at a
        # time, must read).  The copies read far fewer bytes than that, from a
        # working set that sits in the caches, so the model's rate can exceed the
        # HBM peak: it is reported beside the kernel's own floor, and the counters
        # below, where there are any of these kernels, say what binds.
        method = {4: k4_kernel_bytes, 5: k5_method_bytes, 3: k3_kernel_bytes}[dominant](st)
        roofline["method_model_bytes"] = method
        roofline["method_model_frac"] = round(method / (kms * 1e-3) / 1e9 / HBM_PEAK_GBS, 3)
        roofline["binding"] = stored_counters(kname, args.workload)
    if args.calibration_copy_mib > 0:  # a copy of known size for the counter runs
        a = torch.empty(args.calibration_copy_mib << 18, dtype=torch.float32, device=dev)
        torch.empty_like(a).copy_(a)
        torch.cuda.synchronize()

    cpu = None
    if not args.no_cpu:
        cpu = cpu_baseline(g, ks, {k: int(ref[k].sum()) for k in ks}, args.cpu_seconds)

    value = g.m / (ms_per_step * 1e-3)
    line = {
        "metric": "arcs censused/sec",
        "value": round(value, 1),
        "unit": "arcs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u64",
        "data": "synthetic",
        "config": {"workload": args.workload, "n": g.n, "m": g.m, "mstar": st["mstar"], "k": list(ks),
                   "generator": describe(args.workload)},
        "detail": {f"k{k}": {"census_kernel_ms": round(float(np.mean(kern_ms[k])), 3),
                             "build_ms": round(float(np.mean(build_ms[k])), 3),
                             "connected_sets": int(ref[k].sum())} for k in ks},
        "checks": checks,
        "roofline": roofline,
        "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)


def kernel_name(k: int, scheme: int, n: int, m: int, sizes: int) -> str:
    """The kernels between the census events of the largest size k of `sizes`:
    the subgraph copies, the reuse of cores (k = 4 alone on small inputs; k = 5
    of graphs that the copies leave out by their size) or the per-anchor kernel.
    Not told here: k = 5 of a graph with more triangles than the copies have room
    for, counted by the reuse of cores too."""
    if k > 3 and scheme != 1:
        return f"k{k}_kernel"
    if k == 4 and sizes == 1 and n <= 5120 and m <= 5120:
        return "kr_kernel<4>"
    if k == 5 and (n > 65536 or m > 1 << 20 or 3 * m > n * (n - 1)):
        return "kr_kernel<5>"
    return f"copies<{k}>"


TRAFFIC_DIR = os.path.join(ROOT, "profiles")
CENSUS_SRC = [os.path.join(ROOT, "paper_1203_3415_amd", "csrc", f)
              for f in ("census.hip", "counts.h", "counts.hip", "copies5.hip")]


def _src_digest() -> str:
    """SHA-256 of the census source with comments and blank lines removed, so
    that the stored traffic stays valid across comment edits only."""
    import hashlib
    import re
    code = []
    for path in CENSUS_SRC:
        with open(path) as f:
            code += [re.sub(r"//.*$", "", line).rstrip() for line in f]
    return hashlib.sha256("\n".join(x for x in code if x).encode()).hexdigest()


def _traffic_file(kname: str, workload: str) -> str:
    safe = kname.replace("<", "").replace(">", "")
    return os.path.join(TRAFFIC_DIR, f"traffic_{safe}_{workload}.json")


def stored_traffic(kname: str, workload: str):
    """HBM bytes per launch from the committed counter runs, or None when
    there are none or the census kernels changed since they were taken."""
    path = _traffic_file(kname, workload)
    if not os.path.exists(path):
        return None
    with open(path) as f:
        rec = json.load(f)
    return rec["bytes_per_launch"] if rec.get("census_src_sha256") == _src_digest() else None


def traffic_from_counters(fetch_csv: str, write_csv: str, kname: str, workload: str, copy_mib: int):
    """Turn a FETCH_SIZE run and a WRITE_SIZE run (rocprofv3 --pmc, csv) of
    `bench.py --calibration-copy-mib N` into bytes per launch of the kernel:
    each counter is scaled by what it reads for the copy of N MiB (which
    reads and writes exactly N MiB), then averaged over the kernel's
    dispatches.  Writes the record next to the other profile summaries."""
    import csv
    stem = kname.split("<")[0]
    kk = kname[len(stem):]  # "<4>" or ""

    def load(path, counter):
        per = {}
        for r in csv.DictReader(open(path)):
            if r["Counter_Name"] != counter:
                continue
            key = (r["Kernel_Name"], r["Dispatch_Id"])
            per[key] = per.get(key, 0.0) + float(r["Counter_Value"]) * 1024.0  # KiB -> bytes
        kern = [v for (name, _), v in per.items() if f"{stem}<{kk[1:-1]}," in name] if kk else \
            [v for (name, _), v in per.items() if f"{stem}<" in name]
        copies = [v for (name, _), v in per.items() if "copyBuffer" in name or "copy" in name.lower()]
        return kern, max(copies) if copies else None

    kf, cf = load(fetch_csv, "FETCH_SIZE")
    kw, cw = load(write_csv, "WRITE_SIZE")
    ref = float(copy_mib << 20)
    sf, sw = ref / cf, ref / cw
    rec = {"kernel": kname, "workload": workload, "dispatches": [len(kf), len(kw)],
           "fetch_bytes_raw": float(np.mean(kf)), "write_bytes_raw": float(np.mean(kw)),
           "copy_mib": copy_mib, "fetch_scale": sf, "write_scale": sw,
           "bytes_per_launch": float(np.mean(kf)) * sf + float(np.mean(kw)) * sw,
           "census_src_sha256": _src_digest()}
    os.makedirs(TRAFFIC_DIR, exist_ok=True)
    with open(_traffic_file(kname, workload), "w") as f:
        json.dump(rec, f, indent=1)
    print(json.dumps(rec))


def _counters_file(kname: str, workload: str) -> str:
    safe = kname.replace("<", "").replace(">", "")
    return os.path.join(TRAFFIC_DIR, f"counters_{safe}_{workload}.json")


def stored_counters(kname: str, workload: str):
    """Occupancy, issue and cache figures of the kernel from the committed
    counter runs (see counters_from_csv), or None when there are none or the
    census kernels changed since they were taken."""
    path = _counters_file(kname, workload)
    if not os.path.exists(path):
        return None
    with open(path) as f:
        rec = json.load(f)
    if rec.get("census_src_sha256") != _src_digest():
        return None
    return rec["derived"]


def counters_from_csv(dirs: dict, kname: str, workload: str):
    """Per-launch averages of the kernel's counters from rocprofv3 --pmc csv
    runs (dirs: pass name -> counter_collection.csv), and the figures derived
    from them: L2 hit rate, the fractions of resident wave-cycles issuing
    VALU / LDS / vector-memory instructions or waiting, LDS bank conflicts."""
    import csv
    stem, kk = kname.split("<")[0], kname[len(kname.split("<")[0]):]
    vals, copy_vals = {}, {}
    for _, path in dirs.items():
        per, cper = {}, {}
        for r in csv.DictReader(open(path)):
            name = r["Kernel_Name"]
            key = (r["Counter_Name"], r["Dispatch_Id"])
            if "copy" in name.lower():  # the reference copy of --calibration-copy-mib
                cper[key] = cper.get(key, 0.0) + float(r["Counter_Value"])
            if not ((f"{stem}<{kk[1:-1]}," in name) if kk else (f"{stem}<" in name)):
                continue
            per[key] = per.get(key, 0.0) + float(r["Counter_Value"])
        by = {}
        for (cn, _), v in per.items():
            by.setdefault(cn, []).append(v)
        for cn, vs in by.items():
            vals[cn] = float(np.mean(vs))
        for (cn, _), v in cper.items():
            copy_vals[cn] = max(copy_vals.get(cn, 0.0), v)
    d = {}
    # bytes from the request counts by size (no calibration needed): reads of
    # 32, 64 and 128 bytes, writes of 64 bytes and the rest of 32 bytes
    def by_size(v):
        out = {}
        if all(c in v for c in ("TCC_EA0_RDREQ_32B_sum", "TCC_EA0_RDREQ_64B_sum", "TCC_EA0_RDREQ_128B_sum")):
            out["read_bytes_by_request_size"] = (32 * v["TCC_EA0_RDREQ_32B_sum"] + 64 * v["TCC_EA0_RDREQ_64B_sum"] +
                                                 128 * v["TCC_EA0_RDREQ_128B_sum"])
            if "TCC_EA0_RDREQ_sum" in v:
                out["read_requests_other_sizes"] = v["TCC_EA0_RDREQ_sum"] - (
                    v["TCC_EA0_RDREQ_32B_sum"] + v["TCC_EA0_RDREQ_64B_sum"] + v["TCC_EA0_RDREQ_128B_sum"])
        if "TCC_EA0_WRREQ_sum" in v and "TCC_EA0_WRREQ_64B_sum" in v:
            out["write_bytes_by_request_size"] = (64 * v["TCC_EA0_WRREQ_64B_sum"] +
                                                  32 * (v["TCC_EA0_WRREQ_sum"] - v["TCC_EA0_WRREQ_64B_sum"]))
        return out
    d.update(by_size(vals))
    if copy_vals:
        d.update({"copy_" + k2: v2 for k2, v2 in by_size(copy_vals).items()})
    if "TCC_HIT_sum" in vals and "TCC_MISS_sum" in vals:
        d["l2_hit_rate"] = round(vals["TCC_HIT_sum"] / max(1.0, vals["TCC_HIT_sum"] + vals["TCC_MISS_sum"]), 3)
    if vals.get("SQ_WAVE_CYCLES", 0) > 0:
        # each SQ_ACTIVE_INST_* and SQ_WAIT_INST_ANY count wave-cycles like
        # SQ_WAVE_CYCLES, so their ratios are the fractions of the resident
        # waves' time spent issuing that kind of instruction, or waiting
        wc = vals["SQ_WAVE_CYCLES"]
        for cn, nm in (("SQ_ACTIVE_INST_VALU", "valu_issue_frac"), ("SQ_ACTIVE_INST_LDS", "lds_issue_frac"),
                       ("SQ_ACTIVE_INST_VMEM", "vmem_issue_frac"), ("SQ_WAIT_INST_ANY", "wait_frac")):
            if cn in vals:
                d[nm] = round(vals[cn] / wc, 3)
    if "SQ_INSTS_LDS" in vals and "SQ_LDS_BANK_CONFLICT" in vals:
        d["lds_bank_conflict_cycles_per_lds_inst"] = round(vals["SQ_LDS_BANK_CONFLICT"] / max(1.0, vals["SQ_INSTS_LDS"]), 3)
    rec = {"kernel": kname, "workload": workload, "counters_per_launch": vals, "derived": d,
           "census_src_sha256": _src_digest()}
    os.makedirs(TRAFFIC_DIR, exist_ok=True)
    with open(_counters_file(kname, workload), "w") as f:
        json.dump(rec, f, indent=1)
    print(json.dumps(rec))


def describe(name):
    return {
        "chunglu_n1e5_k34": "Chung-Lu n=100000 m=1000000 gamma_out=gamma_in=2.1 reciprocity=0.2 seed=2",
        "chunglu_n1e5_k3": "Chung-Lu n=100000 m=1000000 gamma_out=gamma_in=2.1 reciprocity=0.2 seed=2, k=3 alone",
        "chunglu_n1e5_k4": "Chung-Lu n=100000 m=1000000 gamma_out=gamma_in=2.1 reciprocity=0.2 seed=2, k=4 alone",
        "gnm_n1000": "G(n=1000, 5000 arcs) + 10% reciprocated, seed=1",
        "chunglu_n2e4_k5": "Chung-Lu n=20000 m=100000 gamma_out=2.2 gamma_in=2.5 reciprocity=0.1 seed=4",
    }.get(name, name)


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _mean_sd(xs):
    xs = np.asarray(xs, dtype=np.float64)
    return float(xs.mean()), float(xs.std(ddof=1)) if xs.size > 1 else 0.0


def method_ref_timing(g, ks, threads, budget_s):
    """The CPU method reference (the paper's algorithm written out in C, the
    analogue of its Java acc-Motif) timed on the host: the full census on all
    cores when a 1/64 sample predicts it fits the budget, else projected from
    that sample; single thread projected from a 1/64 sample.  Projection =
    build + 64 * (sample - build), the build timed on its own."""
    import oracle
    out, proj_all, proj_one = {}, 0.0, 0.0
    for k in ks:
        oracle.class_table(k)
        oracle.multiplicities(k)

        def timed(fn):
            t = time.perf_counter()
            fn()
            return time.perf_counter() - t
        build1 = timed(lambda: oracle.method_census_sample(g, k, 1 << 40, threads=1))
        s1 = timed(lambda: oracle.method_census_sample(g, k, 64, threads=1))
        buildn = timed(lambda: oracle.method_census_sample(g, k, 1 << 40, threads=threads))
        sn = timed(lambda: oracle.method_census_sample(g, k, 64, threads=threads))
        one = build1 + 64 * max(0.0, s1 - build1)
        alln = buildn + 64 * max(0.0, sn - buildn)
        how = "projected from a 1/64 sample"
        if alln < budget_s:
            alln = timed(lambda: oracle.method_census(g, k, threads=threads))
            how = "full census"
        proj_all += alln
        proj_one += one
        out[f"k{k}"] = {"seconds_all_cores": round(alln, 2), "all_cores": how,
                        "seconds_single_thread": round(one, 2), "single_thread": "projected from a 1/64 sample"}
    return {"value_all_cores": round(g.m / proj_all, 1), "value_single_thread": round(g.m / proj_one, 1),
            "unit": "arcs/s", "detail": out}


def cpu_baseline(g, ks, total_sets, seconds):
    """The oracle (ESU + k! canonical labelling) timed on the host cores on a
    bounded sample: ESU from roots in a seeded random order for a fixed time,
    5 rounds on all cores and 1 round on one thread per k; the rate in
    connected sets per second projects the full census time.  Beside it, the
    CPU method reference (the paper's own algorithm)."""
    import oracle
    threads = _threads()
    roots = np.random.default_rng(12345).permutation(g.n).astype(np.int32)
    per_round = seconds / 6.0
    proj, proj_sd2, proj_one = 0.0, 0.0, 0.0
    sample = {}
    for k in ks:
        oracle.class_table(k)  # table build excluded from timing
        rates = []
        for _ in range(5):
            t = time.perf_counter()
            h = oracle.census_timed(g, k, roots, per_round, threads=threads)
            dt = time.perf_counter() - t
            rates.append(int(h.sum()) / dt)
        t = time.perf_counter()
        h1 = oracle.census_timed(g, k, roots, per_round, threads=1)
        rate1 = int(h1.sum()) / (time.perf_counter() - t)
        mean, sd = _mean_sd(rates)
        tk = total_sets[k] / mean
        proj += tk
        proj_sd2 += (tk * sd / mean) ** 2
        proj_one += total_sets[k] / rate1
        sample[f"k{k}"] = {"sets_per_s": round(mean, 1), "sets_per_s_sd": round(sd, 1),
                           "sets_per_s_single_thread": round(rate1, 1), "projected_seconds": round(tk, 1)}
    value = g.m / proj
    value_sd = value * (proj_sd2 ** 0.5) / proj
    return {"value": round(value, 3), "unit": "arcs/s", "cores": threads, "kind": "oracle",
            "sample": (f"ESU from roots in seeded random order: 5 rounds of {per_round:.1f} s on {threads} threads "
                       f"and 1 round on 1 thread per k; full-census time projected from connected sets/s"),
            "value_sd": round(value_sd, 3), "rounds": 5, "cpu_model": cpu_model(),
            "single_thread": {"value": round(g.m / proj_one, 3), "unit": "arcs/s"},
            "projected_seconds": round(proj, 1), "detail": sample,
            "method_ref": method_ref_timing(g, ks, threads, budget_s=seconds)}


# ------------------------------------------------------- batch & serving ---

def nullmodel_bases(mode: str, count: int):
    """mode 'same': one Chung-Lu base (n=2000, m=8000, exponent 2.3,
    reciprocity 0.05, seed 3), randomised `count` times; mode 'uneven':
    `count`+1 graphs with n uniform in [500, 5000], m = 4n, each its own
    Chung-Lu base (exponent 2.3, reciprocity 0.05), graphs 1..count each
    randomised once.  Randomisation = switches_per_arc * m attempted arc
    switches on the device (motif_null_randomize)."""
    import graphgen as gg
    if mode == "same":
        return [gg.chung_lu(2000, 8000, 2.3, 2.3, 0.05, seed=3)]
    rng = np.random.default_rng(33)
    out = []
    for i in range(count + 1):
        n = int(rng.integers(500, 5001))
        out.append(gg.chung_lu(n, 4 * n, 2.3, 2.3, 0.05, seed=20000 + i))
    return out


def bench_nullmodel(args):
    import torch
    import graphgen as gg
    import paper_1203_3415_amd as pm

    dev = torch.device("cuda:0")
    count, spa = args.null_graphs, args.switch_per_arc
    report = {}

    def timed(fn, reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t) / reps

    for mode in ("same", "uneven"):
        bases = nullmodel_bases(mode, count)
        dbase = [(*pm.to_device(x.out_off, x.out_idx, dev), x.n) for x in bases]
        if mode == "same":
            off, idx, n = dbase[0]
            d = [dbase[0]] + [(off, idx.clone(), n) for _ in range(count)]
        else:
            d = [dbase[0]] + [(o, i.clone(), nn) for (o, i, nn) in dbase[1:]]
        arcs = int(sum(int(t[1].numel()) for t in d))
        # generation alone: the randomisation of graphs 1..count on the device
        fresh = [t[1].clone() for t in d[1:]]

        def regenerate(seed=1000):
            for t, f in zip(d[1:], fresh):
                t[1].copy_(f)
            pm.null_randomize(d[1:], spa, seed)
        regenerate()
        gen_s = timed(lambda: regenerate(), max(1, args.steps // 2))
        # host generator (graphgen's C switcher), for reference: 8 graphs, scaled
        t = time.perf_counter()
        gg.arc_switch_many(bases[0], spa * bases[0].m, np.arange(1000, 1008))
        host_gen_s = (time.perf_counter() - t) / 8 * count
        print(f"[nullmodel] {mode}: {len(d)} graphs, device generation {gen_s * 1e3:.1f} ms "
              f"(host switcher ~{host_gen_s:.1f} s)", file=sys.stderr, flush=True)
        regenerate()
        out = torch.empty((len(d), 199), dtype=torch.int64, device=dev)
        # without --autotune the fused census of a batch runs under the
        # library's batch default for k = 4 (motif.h, motif_set_tuning)
        tuned = pm.autotune(d, 4) if args.autotune else "library batch default"
        for _ in range(args.warmup):
            pm.census_batch(d, 4, out=out)
        timings = {"fused": timed(lambda: pm.census_batch(d, 4, out=out), args.steps)}
        hb = out.cpu().numpy().view(np.uint64).copy()
        plan = pm.BatchPlan(d, 4)
        plan.run()
        timings["graph_replay"] = timed(plan.run, args.steps)
        hp = plan.hists().copy()
        plan.close()
        pm.census_batch_loop(d, 4, out=out)
        timings["loop"] = timed(lambda: pm.census_batch_loop(d, 4, out=out), args.steps)
        hl = out.cpu().numpy().view(np.uint64).copy()
        z = pm.zscores(hb)
        print(f"[nullmodel] {mode}: fused {timings['fused'] * 1e3:.1f} ms, replay "
              f"{timings['graph_replay'] * 1e3:.1f} ms, loop {timings['loop'] * 1e3:.1f} ms", file=sys.stderr,
              flush=True)
        rec = {"graphs": len(d), "arcs_total": arcs,
               "device_generation_ms": round(gen_s * 1e3, 2), "host_generation_s_est": round(host_gen_s, 1),
               "census_graphs_per_s": {kk: round(len(d) / v, 1) for kk, v in timings.items()},
               "census_ms": {kk: round(v * 1e3, 2) for kk, v in timings.items()},
               "identical_fused_replay_loop": bool(np.array_equal(hb, hl) and np.array_equal(hb, hp)),
               "tuning": tuned, "finite_z": int(np.isfinite(z).sum())}
        if mode == "same":
            # the whole job on the device: replicate, randomise, census, z-scores
            off, idx, n = dbase[0]
            hz = torch.empty((count + 1, 199), dtype=torch.int64, device=dev)
            zz = torch.empty(199, dtype=torch.float64, device=dev)
            pm.null_model(off, idx, n, count, 4, spa, 1000, out=hz, z_out=zz)
            job = timed(lambda: pm.null_model(off, idx, n, count, 4, spa, 1000, out=hz, z_out=zz), args.steps)
            hzn = hz.cpu().numpy().view(np.uint64)
            zd = zz.cpu().numpy()
            ok = np.isfinite(pm.zscores(hzn))
            rec["job_ms"] = round(job * 1e3, 2)
            rec["job_graphs_per_s"] = round(len(d) / job, 1)
            rec["job_z_matches_host"] = bool(np.allclose(zd[ok], pm.zscores(hzn)[ok], rtol=1e-12, atol=0))
            rec["job_hists_equal_in_place_ensemble"] = bool(np.array_equal(hzn, hb))
            print(f"[nullmodel] same: whole job {job * 1e3:.1f} ms", file=sys.stderr, flush=True)
        report[mode] = rec
        del d, out, dbase, fresh
        torch.cuda.empty_cache()
    main_mode = report["same"]
    value = main_mode["job_graphs_per_s"]
    line = {"metric": "null-model graphs/sec", "value": value, "unit": "graphs/s",
            "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": main_mode["job_ms"],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u64", "data": "synthetic",
            "config": {"workload": "nullmodel_k4", "k": 4, "switch_attempts_per_arc": spa,
                       "same": "Chung-Lu n=2000 m=8000 exp 2.3 recip 0.05 + randomisations",
                       "uneven": "n uniform in [500,5000], m=4n, each its own Chung-Lu base randomised",
                       "value": "whole job on the device per graph: randomisation + fused census + z-scores"},
            "detail": report}
    print(json.dumps(line), flush=True)


def _serving_graph(j: int, log_m_max: float):
    import graphgen as gg
    r = np.random.default_rng(10000 + j)
    m = int(round(10 ** r.uniform(3, log_m_max)))
    gamma = float(r.uniform(2.1, 2.6))
    recip = float(r.uniform(0, 0.2))
    k = int(r.integers(3, 6))
    if k == 5 and m > 200_000:
        k = int(r.integers(3, 5))
    n = max(10, m // 5)
    return gg.chung_lu(n, m, gamma, gamma, recip, seed=10000 + j), k


def bench_serving(args):
    """Open-loop Poisson arrivals (rate `--rate`/s) of census requests drawn
    from a pool of `--pool` pregenerated graphs: m log-uniform in
    [1e3, 10^serve_log_m_max], n = m/5, Chung-Lu exponent uniform in
    [2.1, 2.6], reciprocity uniform in [0, 0.2], k uniform in {3,4,5} (k = 5
    only for m <= 2e5).  `--serve-warmup` s of arrivals are served but not
    measured, then `--serve-seconds` s are.  A request that arrives while
    `--max-outstanding` are in flight is shed; a shed request counts as an SLO
    miss (infinite latency) in the percentiles over offered requests.
    Latency = arrival -> histogram on the host; every histogram is checked
    against the same graph censused alone (before the run)."""
    import multiprocessing as mp
    import torch
    import paper_1203_3415_amd as pm

    t0 = time.perf_counter()
    with mp.get_context("spawn").Pool(min(16, os.cpu_count() or 1)) as p:  # workers touch no GPU
        pool = p.starmap(_serving_graph, [(j, args.serve_log_m_max) for j in range(args.pool)])
    print(f"[serving] pool of {len(pool)} graphs generated in {time.perf_counter() - t0:.1f} s", file=sys.stderr,
          flush=True)
    # each graph censused alone, through the plain entry point
    alone = []
    for g, k in pool:
        off, idx = pm.to_device(g.out_off, g.out_idx)
        alone.append(pm.census(off, idx, g.n, k))
        del off, idx
    torch.cuda.empty_cache()
    print(f"[serving] alone results in {time.perf_counter() - t0:.1f} s", file=sys.stderr, flush=True)
    rng = np.random.default_rng(5)
    lam, warm, dur = args.rate, args.serve_warmup, args.serve_seconds
    total_t = warm + dur
    arrivals = np.cumsum(rng.exponential(1.0 / lam, size=int(lam * total_t * 2) + 10))
    arrivals = arrivals[arrivals < total_t]
    picks = rng.integers(0, len(pool), size=arrivals.size)
    lat, shed, wrong = {}, set(), 0
    with pm.Server(args.hbm_budget, max_inflight=args.inflight) as srv:
        start = time.perf_counter()
        pending = []
        last_print = [start]

        def reap(block=False):
            nonlocal wrong
            still = []
            for tk2, ta, i in pending:
                try:
                    h = srv.wait(tk2, timeout_us=-1 if block else 0)
                    lat[i] = time.perf_counter() - ta
                    if not np.array_equal(h, alone[picks[i]]):
                        wrong += 1
                except TimeoutError:
                    still.append((tk2, ta, i))
            return still

        for i, (t_arr, pidx) in enumerate(zip(arrivals, picks)):
            now = time.perf_counter() - start
            if t_arr > now:
                time.sleep(t_arr - now)
            pending = reap()
            if time.perf_counter() - last_print[0] > 5.0:
                last_print[0] = time.perf_counter()
                print(f"[serving] t={now:.0f} s: {len(lat)} done, {len(pending)} in flight, {len(shed)} shed",
                      file=sys.stderr, flush=True)
            if len(pending) >= args.max_outstanding:
                shed.add(i)
                continue
            g, k = pool[pidx]
            try:
                tk = srv.submit(g.out_off, g.out_idx, g.n, k)
            except pm.MotifError:
                shed.add(i)
                continue
            pending.append((tk, start + t_arr, i))
        pending = reap(block=True)
        end = time.perf_counter()
        stats = srv.stats()
    measured = [i for i in range(arrivals.size) if arrivals[i] >= warm]
    m_done = [lat[i] for i in measured if i in lat]
    m_shed = sum(1 for i in measured if i in shed)
    # percentiles over offered requests: a shed request is an SLO miss (infinite latency)
    offered = np.array([lat.get(i, np.inf) for i in measured]) * 1e3
    done_t = [arrivals[i] + lat[i] for i in measured if i in lat]
    span = (max(done_t) - warm) if done_t else dur
    line = {"metric": "census requests/sec", "value": round(len(m_done) / max(span, dur), 2), "unit": "req/s",
            "n_gpus": 1, "steps": 1, "warmup": 1, "ms_per_step": round((end - start) * 1e3, 1),
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u64", "data": "synthetic",
            "config": {"workload": "serving", "rate_per_s": lam, "warmup_s": warm, "seconds": dur,
                       "pool": len(pool), "inflight": args.inflight, "max_outstanding": args.max_outstanding,
                       "hbm_budget_bytes": args.hbm_budget, "log10_m_range": [3, args.serve_log_m_max]},
            "detail": {"p50_ms_offered": round(float(np.percentile(offered, 50)), 2) if offered.size else None,
                       "p99_ms_offered": (round(float(np.percentile(offered, 99)), 2)
                                          if offered.size and np.isfinite(np.percentile(offered, 99)) else "inf"),
                       "p50_ms_completed": round(float(np.percentile(m_done, 50)) * 1e3, 2) if m_done else None,
                       "p99_ms_completed": round(float(np.percentile(m_done, 99)) * 1e3, 2) if m_done else None,
                       "offered": len(measured), "completed": len(m_done), "shed": m_shed,
                       "responses_checked": len(lat), "responses_wrong": wrong,
                       "peak_bytes_admitted": stats["peak_bytes"]}}
    print(json.dumps(line), flush=True)


def bench_census6(args):
    """The k = 6 census (connected 4-set anchors) of a small power-law
    digraph: one step = one motif_census6 call (validation, G* build, anchor
    count and list, census, exact division), host-timed; the CPU baseline is
    the oracle's full ESU census of the same graph on all host cores."""
    import torch
    import graphgen as gg
    import paper_1203_3415_amd as pm

    g = gg.chung_lu(300, 700, 2.3, 2.4, 0.2, seed=62)
    dev = torch.device("cuda:0")
    off, idx = pm.to_device(g.out_off, g.out_idx, dev)
    out = torch.empty(pm.NUM_CLASSES6, dtype=torch.int64, device=dev)
    for _ in range(max(1, args.warmup)):  # the first call also builds the class table
        pm.census6(off, idx, g.n, out=out)
    torch.cuda.synchronize()
    ref = out.cpu().numpy().view(np.uint64).copy()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        pm.census6(off, idx, g.n, out=out)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1000.0 / args.steps
    stable = bool(np.array_equal(out.cpu().numpy().view(np.uint64), ref))
    line = {"metric": "arcs censused/sec", "value": round(g.m / (ms * 1e-3), 1), "unit": "arcs/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 3), "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "u64", "data": "synthetic",
            "config": {"workload": "chunglu_n300_k6", "n": g.n, "m": g.m, "k": [6],
                       "generator": "Chung-Lu n=300 m=700 gamma_out=2.3 gamma_in=2.4 reciprocity=0.2 seed=62"},
            "detail": {"k6": {"connected_sets": int(ref.sum()), "classes_seen": int(np.count_nonzero(ref)),
                              "step": "whole motif_census6 call"}},
            "checks": {"stable_across_steps": stable},
            "roofline": None, "cpu_baseline": None}
    if not args.no_cpu:
        import oracle
        threads = _threads()
        t = time.perf_counter()
        d = oracle.census6(g, threads=threads)
        sec = time.perf_counter() - t
        by_code = dict(zip((int(c) for c in pm.class6_codes()[np.flatnonzero(ref)]),
                           (int(v) for v in ref[np.flatnonzero(ref)])))
        line["checks"]["equals_oracle"] = by_code == d
        line["cpu_baseline"] = {"value": round(g.m / sec, 1), "unit": "arcs/s", "cores": threads,
                                "kind": "oracle", "sample": "the full ESU census of the same graph by canonical code",
                                "seconds": round(sec, 2), "cpu_model": cpu_model()}
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="chunglu_n1e5_k34",
                    choices=["chunglu_n1e5_k34", "chunglu_n1e5_k3", "chunglu_n1e5_k4", "gnm_n1000", "chunglu_n2e4_k5",
                             "nullmodel_k4", "serving", "chunglu_n300_k6"])
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--null-graphs", type=int, default=1000)
    ap.add_argument("--switch-per-arc", type=int, default=100, help="arc-switch attempts per arc of each null graph")
    ap.add_argument("--autotune", action="store_true", help="null model: autotune on each ensemble first")
    ap.add_argument("--rate", type=float, default=200.0)
    ap.add_argument("--serve-seconds", type=float, default=30.0)
    ap.add_argument("--serve-warmup", type=float, default=5.0)
    ap.add_argument("--max-outstanding", type=int, default=64)
    ap.add_argument("--serve-log-m-max", type=float, default=6.0)
    ap.add_argument("--pool", type=int, default=512)
    ap.add_argument("--inflight", type=int, default=4)
    ap.add_argument("--hbm-budget", type=int, default=64 << 30)
    ap.add_argument("--calibration-copy-mib", type=int, default=0,
                    help="after the timed steps, copy this many MiB on the device (reference for HBM counters)")
    ap.add_argument("--traffic-from", nargs=2, metavar=("FETCH_CSV", "WRITE_CSV"),
                    help="no GPU: turn two rocprofv3 --pmc csv files into the stored traffic record")
    ap.add_argument("--kernel", default="copies<4>", help="kernel of --traffic-from / --counters-from")
    ap.add_argument("--counters-from", nargs="+", metavar="CSV",
                    help="no GPU: turn rocprofv3 --pmc csv files into the stored counter record")
    args = ap.parse_args()
    if args.counters_from:
        counters_from_csv({str(i): p for i, p in enumerate(args.counters_from)}, args.kernel, args.workload)
        return
    if args.traffic_from:
        traffic_from_counters(args.traffic_from[0], args.traffic_from[1], args.kernel, args.workload,
                              args.calibration_copy_mib)
        return
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) > 1:
        print(json.dumps({"error": "this census runs on one GPU; --gpus must be 1 (multi-GPU sharding is a "
                                   "design note only)"}), flush=True)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        raise SystemExit("bench.py needs a GPU")
    if args.workload == "nullmodel_k4":
        bench_nullmodel(args)
    elif args.workload == "serving":
        bench_serving(args)
    elif args.workload == "chunglu_n300_k6":
        bench_census6(args)
    else:
        bench_census(args)


if __name__ == "__main__":
    main()
