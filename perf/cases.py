"""The workloads this library is timed on: what a program does with it through the Python package.

A case is one evolving graph (an R-MAT base edge set and K update batches, the recipe of the repository's
synthetic inputs) and one operation on it:

  query    one query over a window of snapshots on a resident graph (Graph.query)
  noalloc  the same from a caller that cannot allocate (Graph.query_noalloc)
  batch    many queries answered together, each expanded to its dense values (Graph.query_batch)
  serve    queries submitted to a running server and collected (Server, continuous batching)
  append   the ring advanced by one batch, then a query on the newest snapshots (Graph.append)
  build    the versioned graph built from host edge lists, then one bounds query (Graph, Graph.query_bounds)

The inputs are drawn on the GPU from the seed alone.  Values are uint32 held in int32 tensors.
"""
import math
import random

import numpy as np
import torch

import paper_2502_10579_amd as evq

QUADRANTS = (0.57, 0.19, 0.19)  # the R-MAT recipe of the repository's inputs
INF, SAT = 0xFFFFFFFF, 0xFFFFFFFE
ALGOS = ("sssp", "bfs", "sswp", "ssnp", "viterbi")


def _case(name, op, algo, vertices, edges, snapshots, updates, wmax=100, begin=0, length=None, queries=1):
    """length None: every snapshot.  updates: deletions, and as many additions, per snapshot."""
    c = dict(op=op, algo=algo, vertices=vertices, edges=edges, snapshots=snapshots, updates=updates, wmax=wmax,
             begin=begin, length=snapshots if length is None else length, queries=queries)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest calls: a graph that fits in a cache, where a query is launches and waits.
        _case("query_small_sssp", "query", "sssp", 1 << 12, 32768, 8, 33),
        # A caller under graph capture or in a tight loop, on a graph its scratch holds.
        _case("noalloc_ssnp", "noalloc", "ssnp", 1 << 16, 1 << 20, 32, 500),
        # An odd size on purpose: vertices, snapshots and window are no round numbers.
        _case("query_odd_ssnp", "query", "ssnp", 150001, 2400007, 50, 1203, wmax=1000, begin=7, length=33),
        # The headline: 64 snapshots of a 16.7M-edge graph under light churn, whole window.
        _case("query_mid_sssp", "query", "sssp", 1 << 20, 1 << 24, 64, 10000),
        # The same graph asked about part of its history: a ragged window, hop counts.
        _case("query_mid_bfs_part", "query", "bfs", 1 << 20, 1 << 24, 64, 10000, begin=17, length=37),
        # Heavy churn: about half of the vertices change within the window, so the relaxation dominates.
        _case("query_churn_sssp", "query", "sssp", 1 << 20, 1 << 24, 64, 100000),
        # 128 snapshots (two-word masks, two snapshots per lane), floating-point values.
        _case("query_mid_viterbi", "query", "viterbi", 1 << 20, 1 << 24, 128, 10000),
        # The largest graph: its values exceed a cache slice and its output is 3.4 GB.
        _case("query_large_sswp", "query", "sswp", 1 << 23, 1 << 27, 100, 50000, wmax=1000),
        # An analyst's batch: mixed algorithms, sources and windows, all dense results wanted.
        _case("batch_mixed", "batch", "mixed", 1 << 20, 1 << 24, 64, 10000, queries=16),
        # A burst of requests to the server over a ring of 128 snapshots.
        _case("serve_burst", "serve", "mixed", 1 << 18, 1 << 22, 128, 2500, queries=12),
        # A stream of updates: each new batch is appended and the newest snapshots are asked about.
        _case("append_query_bfs", "append", "bfs", 1 << 22, 1 << 26, 128, 20000, length=16),
        # A history loaded from host memory: the build, then the bounds of one query.
        _case("build_bounds_sssp", "build", "sssp", 1 << 20, 1 << 24, 64, 10000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(("query", "noalloc", "batch", "serve", "append", "build"), (60, 8, 8, 8, 8, 8))[0]
    top = {"query": 1 << 21, "noalloc": 1 << 16, "batch": 1 << 19, "serve": 1 << 18}.get(op, 1 << 20)
    vertices = 1 << rng.randint(10, top.bit_length() - 1) if rng.random() < 0.25 else _log_int(rng, 1 << 10, top)
    edges = int(vertices * rng.uniform(4, 18))
    snapshots = rng.choice((8, 32, 64, 100, 128)) if rng.random() < 0.5 else rng.randint(2, 128)
    # 0.01% to 0.6% of the edges change per snapshot
    updates = max(1, int(edges * math.exp(rng.uniform(math.log(1e-4), math.log(6e-3)))))
    begin, length = 0, snapshots
    if op == "append":
        length = rng.randint(1, snapshots)
    elif rng.random() < 0.5:
        begin = rng.randint(0, snapshots - 1)
        length = rng.randint(1, snapshots - begin)
    many = op in ("batch", "serve")
    return _case(None, op, "mixed" if many else rng.choice(ALGOS), vertices, edges, snapshots, updates,
                 wmax=rng.choice((10, 100, 1000)), begin=begin, length=length,
                 queries=rng.randint(2, 12) if many else 1)


# ------------------------------------------------------------------ inputs


def _rmat(n, case, gen):
    """(n, 3) int32 rows (source, destination, weight) on the GPU."""
    V = case["vertices"]
    a, b, c = QUADRANTS
    out = torch.empty((n, 3), dtype=torch.int32, device="cuda")
    for i in range(0, n, 1 << 24):
        m = min(1 << 24, n - i)
        src = torch.zeros(m, dtype=torch.int32, device="cuda")
        dst = torch.zeros(m, dtype=torch.int32, device="cuda")
        for _ in range(max(1, (V - 1).bit_length())):
            r = torch.rand(m, generator=gen, device="cuda")
            low = r >= a + b
            right = (r >= a + b + c) | ((r >= a) & ~low)
            src.mul_(2).add_(low)
            dst.mul_(2).add_(right)
        out[i:i + m, 0] = src % V
        out[i:i + m, 1] = dst % V
        out[i:i + m, 2] = torch.randint(1, case["wmax"] + 1, (m,), generator=gen, device="cuda", dtype=torch.int32)
    return out


def _events(case, seed):
    """Base edges, K deletion and K addition batches, and one more batch of each (device tensors), and the
    sources of the case's queries (vertices with out-edges)."""
    gen = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    K, u = case["snapshots"], case["updates"]
    base = _rmat(case["edges"], case, gen)
    adds = _rmat((K + 1) * u, case, gen).view(K + 1, u, 3)
    picks = torch.randint(0, case["edges"], ((K + 1) * u,), generator=gen, device="cuda")
    dels = base[picks].view(K + 1, u, 3)
    has = torch.zeros(case["vertices"], dtype=torch.bool, device="cuda")
    has[base[:, 0].long()] = True
    out = torch.nonzero(has).view(-1)
    at = torch.randint(0, out.numel(), (case["queries"],), generator=gen, device="cuda")
    return base, dels, adds, [int(v) for v in out[at].cpu()]


def _host(t):
    return t.cpu().numpy().view(np.uint32)


def _queries(case, sources):
    """The mixed queries of a batch or a burst: the windows are the case's, the sources the seed's."""
    r = random.Random(12345 + case["queries"])
    K, out = case["snapshots"], []
    for s in sources:
        b = r.randint(0, K - 1) if case["op"] == "batch" else 0
        n = min(r.randint(min(25, K), K), K - b)
        out.append((r.choice(ALGOS[:4]), s, b if case["op"] == "batch" else K - n, n))
    return out


def _windows(case):
    if case["queries"] == 1:
        return [case["length"]]
    return [q[3] for q in _queries(case, [0] * case["queries"])]


def prepare(case, seed):
    base, dels, adds, sources = _events(case, seed)
    V, K = case["vertices"], case["snapshots"]
    host = (_host(base), list(_host(dels[:K])), list(_host(adds[:K])))
    st = dict(case=case, source=sources[0])
    if case["op"] == "build":
        return dict(st, host=host)
    st["out"] = [torch.empty((V, n), dtype=torch.int32, device="cuda") for n in _windows(case)]
    if case["op"] == "append":  # two batches in turn, each undoing the other, so that every append changes edges
        d, a = _host(dels[K]), _host(adds[K])
        st.update(batches=[(d, a), (a, d)], turn=0)
    del base, dels, adds
    st["graph"] = evq.Graph(V, *host)
    if case["op"] in ("batch", "serve"):
        st["queries"] = _queries(case, sources)
    if case["op"] == "serve":
        st["server"] = evq.Server(st["graph"], mode="batch")
    return st


def run(state):
    case, op = state["case"], state["case"]["op"]
    if op == "build":
        with evq.Graph(case["vertices"], *state["host"]) as g:
            return g.query_bounds(case["algo"], state["source"], case["begin"], case["length"])
    g, out = state["graph"], state["out"]
    if op == "query":
        return g.query(case["algo"], state["source"], case["begin"], case["length"], out=out[0])
    if op == "noalloc":
        return g.query_noalloc(case["algo"], state["source"], case["begin"], case["length"], out=out[0])
    if op == "append":
        g.append(*state["batches"][state["turn"]])
        state["turn"] ^= 1
        return g.query(case["algo"], state["source"], g.first + g.K - case["length"], case["length"], out=out[0])
    if op == "batch":
        for r, o in zip(g.query_batch(state["queries"]), out):
            r.expand(out=o)
            r.free()
        return out
    place = {state["server"].submit(a, s, n): i for i, (a, s, _, n) in enumerate(state["queries"])}
    while place:
        for c in state["server"].poll(wait_ms=1000):
            if c["status"] != 0:
                raise RuntimeError("a served query failed with status %d" % c["status"])
            c["result"].expand(out=out[place.pop(c["ticket"])])
            c["result"].free()
    return out


def work(case):
    """Each edge read once (destination and weight; a changing edge its source, mask and place among the
    changing ones too), each value written once; a relaxation of an edge is two operations."""
    V, E, K = case["vertices"], case["edges"], case["snapshots"]
    words = 1 if K <= 64 else 2
    changing = 2 * K * case["updates"]
    values = 4 * V * sum(_windows(case))
    read = 8 * E + (12 + 8 * words) * changing + 8 * V
    if case["op"] == "build":  # the events in, the versioned graph out, then the query reads it
        return {"bytes": 12 * (E + changing) + (8 + 8 * words) * E + read + 8 * V, "flops": 2 * E}
    if case["op"] == "append":  # every edge and its mask in and out, then the query reads them
        return {"bytes": 2 * (8 + 8 * words) * E + 24 * case["updates"] + read + values, "flops": 2 * E}
    algos = 1 if case["queries"] == 1 else len({q[0] for q in _queries(case, [0] * case["queries"])})
    return {"bytes": read + values, "flops": 2 * E * (algos if case["queries"] > 1 else 1)}


# ------------------------------------------------------------------ the values, from torch alone


def _presence(case, base, dels, adds):
    """Distinct triples (source, destination, weight) and, after each batch, which of them are present."""
    V, W = case["vertices"], case["wmax"] + 1

    def key(t):
        t = t.long()
        return (t[:, 0] * V + t[:, 1]) * W + t[:, 2]

    keys = torch.unique(torch.cat([key(base), key(adds.reshape(-1, 3))]))
    now = torch.zeros(keys.numel(), dtype=torch.bool, device="cuda")
    now[torch.searchsorted(keys, key(base))] = True
    snaps = []
    for d, a in zip(dels, adds):
        now = now.clone()
        now[torch.searchsorted(keys, key(d))] = False  # deletions are drawn from the base: each is among the keys
        now[torch.searchsorted(keys, key(a))] = True
        snaps.append(now)
    pair = keys // W
    return (pair // V, pair % V, keys % W), snaps


def _solve(algo, V, edges, present, source):
    """Values on one edge set by rounds over all edges, in 64 bits, as int32 bit patterns."""
    src, dst, w = (e[present] for e in edges)
    if algo == "viterbi":  # defined as single floats: each step divides in double and rounds once
        val = torch.zeros(V, dtype=torch.float32, device="cuda")
        val[source] = 1.0
    else:
        val = torch.full((V,), 0 if algo == "sswp" else INF, dtype=torch.int64, device="cuda")
        val[source] = INF if algo == "sswp" else 0
    while True:
        x = val[src]
        if algo == "viterbi":
            q = x.double() / w.double()
            c = torch.where(q < 2.0 ** -126, 0.0, q).float()
        elif algo == "sswp":
            c = torch.minimum(x, w)
        elif algo == "ssnp":
            c = torch.maximum(x, w)
        else:
            c = torch.where(x == INF, INF, torch.clamp(x + (w if algo == "sssp" else 1), max=SAT))
        new = val.scatter_reduce(0, dst, c, "amax" if algo in ("sswp", "viterbi") else "amin")
        if torch.equal(new, val):
            break
        val = new
    return val.view(torch.int32) if algo == "viterbi" else torch.where(val > 0x7FFFFFFF, val - (1 << 32), val).int()


def exact(case, seed):
    K, V = case["snapshots"], case["vertices"]
    solves = 2 if case["op"] == "build" else sum(_windows(case))
    if case["edges"] * solves > 3e8:
        return None
    base, dels, adds, sources = _events(case, seed)
    n = K + (1 if case["op"] == "append" else 0)
    edges, snaps = _presence(case, base, dels[:n], adds[:n])
    if case["op"] == "build":
        window = torch.stack(snaps[case["begin"]:case["begin"] + case["length"]])
        return tuple(_solve(case["algo"], V, edges, p, sources[0]) for p in (window.all(0), window.any(0)))
    if case["queries"] > 1:
        asked = _queries(case, sources)
    else:
        first = n - case["length"] if case["op"] == "append" else case["begin"]
        asked = [(case["algo"], sources[0], first, case["length"])]
    got = [torch.stack([_solve(a, V, edges, snaps[b + i], s) for i in range(m)], 1) for a, s, b, m in asked]
    return got if case["queries"] > 1 else got[0]
