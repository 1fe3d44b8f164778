"""Performance cases of the framework: what its users run, through the public binding.

A user counts graphlets: builds the count table of a graph under a colouring
(``Table``, ``build_batch`` for many small ones, ``Table16`` for k above 8), then
draws colourful treelets from it and classifies them (``sample``, ``classify``,
``ags``, or many such requests at once through ``Server``). The cases cover each of
these over its range of sizes:

* build     graph and colouring in, table out; the pass ends with the level-k records
            (every stored k-treelet count) and the totals t and t_j. ``lam`` > 0 draws the
            colouring under the biased law first.
* batch     many small uneven graphs in one call; level-k records and totals of each.
* build16   the sparse-record build for k above 8; level-k records and total.
* sample    uniform (shape -1) or shape-restricted samples from a resident table, and
            their classes.
* ags       adaptive graphlet sampling on a resident table.
* serve     a burst of requests to a server over resident tables, until all are answered.

Graphs are made on the GPU from the seed: Erdos-Renyi (er), Chung-Lu with a power-law
weight sequence (cl) and preferential attachment (ba), the families of the benchmark.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2009_03052_amd as scc

ROOTINGS = {"zero": scc.ROOT_ZERO, "all": scc.ROOT_ALL, "balanced": scc.ROOT_BALANCED}
# rooted treelet shapes on h nodes, h = 0..10
ROOTED = (0, 1, 1, 2, 4, 9, 20, 48, 115, 286, 719)


def listed():
    return [
        # the smallest build in use: a graph of a few thousand vertices, every rooting kept; bound by launches
        {"name": "build-er-2k-k4-all", "op": "build", "graph": "er", "n": 2000, "m": 8000, "gamma": 0.0, "wmax": 0.0,
         "k": 4, "rooting": "all", "lam": 0.0, "vlc": False},
        # one of the many colourings that an estimate averages over, on a graph of 5 million edges
        {"name": "build-cl-500k-k7", "op": "build", "graph": "cl", "n": 500_000, "m": 5_000_000, "gamma": 2.2,
         "wmax": 2.5e4, "k": 7, "rooting": "zero", "lam": 0.0, "vlc": False},
        # the middle size: a hub-dominated social graph at k = 6
        {"name": "build-cl-1m-k6", "op": "build", "graph": "cl", "n": 1_000_000, "m": 10_000_000, "gamma": 2.1,
         "wmax": 5e4, "k": 6, "rooting": "zero", "lam": 0.0, "vlc": False},
        # round skipping under a biased colouring, as chosen to save memory on larger graphs
        {"name": "build-cl-2m-k7-balanced", "op": "build", "graph": "cl", "n": 2_000_003, "m": 30_000_001,
         "gamma": 2.4, "wmax": 1e5, "k": 7, "rooting": "balanced", "lam": 0.05, "vlc": False},
        # the largest build: 60 million edges at k = 8, an 85 GB table
        {"name": "build-cl-4m-k8", "op": "build", "graph": "cl", "n": 4_000_000, "m": 60_000_000, "gamma": 2.3,
         "wmax": 2e5, "k": 8, "rooting": "zero", "lam": 0.0, "vlc": False},
        # thirty-two uneven graphs of a collection in one call
        {"name": "batch-32-k5to7", "op": "batch", "count": 32, "n_lo": 1000, "n_hi": 100_000, "draw": 5},
        # a sparse graph above k = 8
        {"name": "build16-cl-64k-k10", "op": "build16", "n": 65_536, "m": 131_072, "gamma": 2.5, "wmax": 40.0, "k": 10},
        # the smallest sampling request: a thousand samples and their classes
        {"name": "sample-1k-k6", "op": "sample", "n": 1_000_000, "m": 10_000_000, "gamma": 2.1, "wmax": 5e4, "k": 6,
         "rooting": "zero", "vlc": False, "shape": -1, "samples": 1000},
        # the bulk: five million uniform samples and their classes at k = 8
        {"name": "sample-5m-k8", "op": "sample", "n": 2_000_000, "m": 30_000_000, "gamma": 2.3, "wmax": 1e5, "k": 8,
         "rooting": "zero", "vlc": False, "shape": -1, "samples": 5_000_000},
        # samples of one shape from a table kept with variable-length counts
        {"name": "sample-100k-k7-shape-vlc", "op": "sample", "n": 1_000_000, "m": 10_000_000, "gamma": 2.2,
         "wmax": 5e4, "k": 7, "rooting": "zero", "vlc": True, "shape": 5, "samples": 99_991},
        # adaptive sampling in twenty rounds
        {"name": "ags-20x100k-k7", "op": "ags", "n": 2_000_000, "m": 30_000_000, "gamma": 2.4, "wmax": 1e5, "k": 7,
         "cbar": 1000, "round": 100_000, "rounds": 20},
        # a burst of requests of mixed sizes on three resident tables
        {"name": "serve-16-on-3-k7", "op": "serve", "tables": 3, "n": 1_000_000, "m": 15_000_000, "k": 7,
         "requests": 16, "lo": 1000, "hi": 1_000_000, "draw": 31},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm, mean degrees from 6 to 30."""
    op = rng.choice(["build", "build", "build", "build", "sample", "sample", "sample", "batch", "build16", "ags", "serve"])
    if op == "build":
        n = _log_int(rng, 2000, 2_000_000)
        k = rng.randint(4, 8)
        rooting = rng.choice(["zero", "zero", "zero", "all", "balanced"])
        if rooting == "all" and k > 6:
            n = min(n, 400_000 + n % 1000)
        m = int(n * rng.uniform(3, 15))
        graph = "er" if n < 50_000 and rng.random() < 0.5 else "cl"
        cl = graph == "cl"
        return {"op": op, "graph": graph, "n": n, "m": m, "gamma": round(rng.uniform(2.1, 2.8), 2) if cl else 0.0,
                "wmax": float(int(n * rng.uniform(0.02, 0.05))) if cl else 0.0, "k": k, "rooting": rooting,
                "lam": round(rng.uniform(0.02, 0.1), 3) if rng.random() < 0.2 else 0.0, "vlc": rng.random() < 0.2}
    if op == "batch":
        return {"op": op, "count": _log_int(rng, 4, 32), "n_lo": 1000, "n_hi": _log_int(rng, 10_000, 100_000),
                "draw": rng.randint(0, 1 << 20)}
    if op == "build16":
        k = rng.randint(9, 11)
        n = _log_int(rng, 2000, {9: 65_536, 10: 40_000, 11: 8000}[k])
        return {"op": op, "n": n, "m": int(n * rng.uniform(1.5, 2.0)), "gamma": round(rng.uniform(2.4, 2.8), 2),
                "wmax": float(rng.randint(20, 40)), "k": k}
    if op == "sample":
        n = _log_int(rng, 10_000, 2_000_000)
        k = rng.randint(4, 8)
        rooting = rng.choice(["zero", "zero", "all" if k < 7 else "zero", "balanced"])
        shape = rng.choice([-1, -1, 1])  # shape 1 exists from k = 4 on
        return {"op": op, "n": n, "m": int(n * rng.uniform(6, 15)), "gamma": round(rng.uniform(2.1, 2.8), 2),
                "wmax": float(int(n * rng.uniform(0.02, 0.05))), "k": k, "rooting": rooting,
                "vlc": rng.random() < 0.25, "shape": shape, "samples": _log_int(rng, 1000, 5_000_000)}
    if op == "ags":
        n = _log_int(rng, 20_000, 1_000_000)
        return {"op": op, "n": n, "m": int(n * rng.uniform(6, 15)), "gamma": round(rng.uniform(2.2, 2.8), 2),
                "wmax": float(int(n * rng.uniform(0.02, 0.05))), "k": rng.randint(5, 7), "cbar": rng.choice([300, 1000]),
                "round": _log_int(rng, 1000, 100_000), "rounds": rng.randint(5, 20)}
    n = _log_int(rng, 50_000, 1_000_000)
    return {"op": op, "tables": rng.randint(1, 3), "n": n, "m": int(n * rng.uniform(6, 15)), "k": rng.randint(5, 7),
            "requests": rng.randint(4, 16), "lo": 1000, "hi": _log_int(rng, 20_000, 1_000_000),
            "draw": rng.randint(0, 1 << 20)}


# ---- inputs -------------------------------------------------------------------------------------


def _generator(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + salt * 7919 + 1) & 0x7FFFFFFFFFFFFFFF)
    return g


def _graph(n, key):
    """The device graph of the distinct undirected edges with keys lo * n + hi."""
    lo, hi = key // n, key % n
    arcs = torch.cat([key, hi * n + lo]).sort().values
    row = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(arcs // n, minlength=n), 0, out=row[1:])
    return scc.DeviceGraph(row.cpu(), (arcs % n).to(torch.int32).cpu())


def _distinct(n, m, g, pairs):
    """m distinct loop-free edges out of what pairs(count) draws."""
    have = torch.zeros(0, dtype=torch.int64, device="cuda")
    while have.numel() < m:
        a, b = pairs(int((m - have.numel()) * 1.15) + 256)
        lo, hi = torch.minimum(a, b), torch.maximum(a, b)
        have = torch.unique(torch.cat([have, (lo * n + hi)[lo != hi]]))
    if have.numel() > m:
        have = have[torch.randperm(have.numel(), generator=g, device="cuda")[:m]].sort().values
    return have


def _erdos_renyi(n, m, g):
    return _graph(n, _distinct(n, m, g, lambda c: torch.randint(0, n, (2, c), generator=g, device="cuda").unbind(0)))


def _chung_lu(n, m, gamma, wmax, g):
    """Weights wmax * (1 + i / i0)^(-1 / (gamma - 1)), i0 so that they sum to 2 m."""
    i = torch.arange(n, dtype=torch.float64, device="cuda")
    lo, hi = 1e-6, 1e12
    for _ in range(60):
        mid = math.sqrt(lo * hi)
        total = float((wmax * (1 + i / mid).pow(-1 / (gamma - 1))).sum())
        lo, hi = (mid, hi) if total < 2 * m else (lo, mid)
    cum = (wmax * (1 + i / lo).pow(-1 / (gamma - 1))).cumsum(0)
    name = torch.randperm(n, generator=g, device="cuda")

    def end(c):
        x = torch.rand(c, dtype=torch.float64, generator=g, device="cuda") * cum[-1]
        return name[torch.searchsorted(cum, x).clamp_(max=n - 1)]

    return _graph(n, _distinct(n, m, g, lambda c: (end(c), end(c))))


def _preferential(n, d, g):
    """Each vertex from d on links to d ends of earlier edges (position 2e: the new vertex, 2e + 1: a copy of
    an earlier position); duplicates merged."""
    edges = (n - d) * d
    e = torch.arange(edges, dtype=torch.int64, device="cuda")
    to = torch.empty(2 * edges, dtype=torch.int64, device="cuda")
    to[0::2] = 2 * e
    to[1::2] = (torch.rand(edges, dtype=torch.float64, generator=g, device="cuda") * (2 * e + 1)).long()
    for _ in range(64):
        nxt = to[to]
        if torch.equal(nxt, to):
            break
        to = nxt
    a, b = e // d + d, to[1::2] // 2 // d + d
    b = torch.where(a == b, e % d, b)  # a self copy links to one of the first d vertices
    return _graph(n, torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b)))


def _make_graph(c, g):
    return _erdos_renyi(c["n"], c["m"], g) if c.get("graph") == "er" else _chung_lu(c["n"], c["m"], c["gamma"], c["wmax"], g)


def _colors(n, k, g):
    return torch.randint(0, k, (n,), dtype=torch.uint8, generator=g, device="cuda")


def _batch_sizes(case):
    """(family, n, mean degree, k) of each graph of a batch."""
    rng = random.Random(case["draw"])
    return [("er" if i % 2 == 0 else "ba", _log_int(rng, case["n_lo"], case["n_hi"]), 4 + i % 17, 5 + (16 + i) % 3)
            for i in range(case["count"])]


def _requests(case):
    """(table, samples, classify, seed) of each sampling request, and the round sizes of each table's AGS session."""
    rng = random.Random(case["draw"])
    reqs = [(rng.randrange(case["tables"]), _log_int(rng, case["lo"], case["hi"]), rng.random() < 0.5,
             rng.randrange(1 << 30)) for _ in range(case["requests"])]
    return reqs, [[_log_int(rng, case["lo"], case["hi"] / 4) for _ in range(2)] for _ in range(case["tables"])]


def prepare(case, seed):
    op, g = case["op"], _generator(seed)
    s = {"case": case, "seed": int(seed) & 0x7FFFFFFF}
    if op == "batch":
        s["instances"] = []
        for i, (family, n, d, k) in enumerate(_batch_sizes(case)):
            graph = _erdos_renyi(n, n * d // 2, g) if family == "er" else _preferential(n, max(1, d // 2), g)
            s["instances"].append((graph, _colors(n, k, g), k))
        return s
    if op == "serve":
        k = case["k"]
        tables = []
        for i in range(case["tables"]):
            graph = _chung_lu(case["n"], case["m"], (2.1, 2.4, 2.8)[i], case["n"] * 0.05, g)
            tables.append(scc.Table(graph, _colors(graph.n, k, g), k))
        s["requests"], s["rounds"] = _requests(case)
        s["server"] = scc.Server(tables, hbm_budget=1 << 30, small_request=1 << 14, small_step=1 << 16)
        return s
    graph = _make_graph(case, g)
    colors = _colors(graph.n, case["k"], g)
    if op in ("build", "build16"):
        s["graph"], s["colors"] = graph, colors
    else:
        s["table"] = scc.Table(graph, colors, case["k"], rooting=ROOTINGS[case.get("rooting", "zero")],
                               vlc=case.get("vlc", False))
    return s


# ---- one pass -----------------------------------------------------------------------------------


def _words(values):
    """Unsigned 128-bit integers as int64 words, low words first."""
    m = (1 << 64) - 1
    return np.array([[v & m, v >> 64 & m] for v in values], dtype=np.uint64).view(np.int64)


def _most_counts(n, k, rooting, lam=0.0):
    """Room for the level-k counts of n vertices: every shape at every vertex that roots one."""
    if rooting == "balanced":
        return n * (scc.num_unrooted(k) - 1)
    roots = n if rooting == "all" else n * (1 - (k - 1) * lam if lam > 0 else 1 / k)
    return ROOTED[k] * min(n, int(roots + 6 * math.sqrt(n)) + 1)


def _level(off, entries, room):
    """The level's offsets and its entries at the head of buffers of a fixed size."""
    return (off, *(torch.nn.functional.pad(x, (0, 0) * (x.dim() - 1) + (0, room - x.shape[0])) for x in entries))


def _summary(t):
    total, shapes = t.totals()
    return _words([total, t.star_count()] + shapes)


def run(state):
    case, seed = state["case"], state["seed"]
    op = case["op"]
    if op == "build":
        g, k = state["graph"], case["k"]
        colors = scc.color_biased(g.n, k, case["lam"], seed) if case["lam"] > 0 else state["colors"]
        t = scc.Table(g, colors, k, rooting=ROOTINGS[case["rooting"]], vlc=case["vlc"])
        off, *entries = t.export_level(k, to_host=False)
        out = (*_level(off, entries, _most_counts(g.n, k, case["rooting"], case["lam"])), _summary(t))
        t.close()
        return out
    if op == "build16":
        t = scc.Table16(state["graph"], state["colors"], case["k"])
        off, *entries = t.export_words(case["k"], 2, to_host=False)
        out = (*_level(off, entries, _most_counts(case["n"], case["k"], "zero")), _words([t.total()]))
        t.close()
        return out
    if op == "batch":
        tables, _ = scc.build_batch(state["instances"])
        off, *entries = (torch.cat(p) for p in zip(*(t.export_level(t.k, to_host=False) for t in tables)))
        room = sum(_most_counts(g.n, k, "zero") for g, _, k in state["instances"])
        out = (*_level(off, entries, room), np.concatenate([_summary(t) for t in tables]))
        for t in tables:
            t.close()
        return out
    if op == "sample":
        t = state["table"]
        verts, parent = t.sample(case["samples"], seed=seed, shape=case["shape"])
        code, cls = t.classify(verts)
        return verts, parent, code, cls
    if op == "ags":
        return state["table"].ags(case["cbar"], case["round"], case["round"] * case["rounds"], seed)
    server = state["server"]
    sessions = [server.ags_open(i, 1000, seed + i) for i in range(case["tables"])]
    ids = [server.submit(t, n, seed=seed ^ q, classify=c) for t, n, c, q in state["requests"]]
    rounds = [server.submit(i, n, session=s) for i, s in enumerate(sessions) for n in state["rounds"][i]]
    out = []
    for rid in ids:
        r = server.wait(rid)
        out.append([r[f] for f in ("verts", "parent", "cls") if r[f] is not None])
        server.release(rid)
    for rid in rounds:
        server.wait(rid, copy=False)
        server.release(rid)
    return out, [server.ags_result(s, i, cap=2) for i, s in enumerate(sessions)]


# ---- what a pass cannot do without --------------------------------------------------------------


def _csr_bytes(n, m):
    return 8 * (n + 1) + 8 * m + n


def _table_counts(n, k, rooting):
    """Stored counts of a full table: h-node shapes times colour sets that hold the root's colour, at each vertex."""
    low = sum(ROOTED[h] * math.comb(k - 1, h - 1) for h in range(2, k - (rooting == "balanced")))
    return n * (low + ROOTED[k] * (1 / k if rooting == "zero" else 0.4 if rooting == "balanced" else 1))


def work(case):
    """Inputs read once, results written once: for a build the graph, the colours and the stored counts (10 bytes
    each, at their number in a well-connected graph) and one multiply-add per edge and stored count below level
    k; for samples the rows and classes written and a 64-byte line for each of the two draws of each step."""
    op = case["op"]
    if op in ("build", "batch"):
        parts = ([(n, n * d // 2, k, "zero") for _, n, d, k in _batch_sizes(case)] if op == "batch"
                 else [(case["n"], case["m"], case["k"], case["rooting"])])
        counts = [_table_counts(n, k, r) for n, _, k, r in parts]
        return {"bytes": sum(_csr_bytes(n, m) + 10 * c for (n, m, _, _), c in zip(parts, counts)),
                "flops": sum(2 * 2 * m / n * c for (n, m, _, _), c in zip(parts, counts))}
    if op == "build16":
        # records of sparse graphs grow about 2.5 times a level
        counts = case["n"] * 2.5 ** (case["k"] - 1)
        return {"bytes": _csr_bytes(case["n"], case["m"]) + 24 * counts, "flops": 4 * counts}
    k = case["k"]
    if op == "sample":
        n = case["samples"]
    elif op == "ags":
        n = case["round"] * case["rounds"]
    else:
        reqs, rounds = _requests(case)
        n = sum(r[1] for r in reqs) + sum(map(sum, rounds))
    return {"bytes": n * (5 * k + 8 + 128 * (k - 1)), "flops": 0}


def exact(case, seed):
    """None: every output is a whole number (counts, vertices, classes) and has to be equal. The only floating
    ones, the class weights of adaptive sampling, follow in 64 bits from the whole numbers of the rounds that the
    sampler itself draws."""
    return None
