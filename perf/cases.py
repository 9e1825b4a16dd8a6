"""The work that a user of this package has it do, as timed cases.

A case is one pass through public entry points of ``paper_2001_06770_amd``:
a single query, a batch (cohort or lanes mode), a round of served queries, a
query without device allocations, a new granularity alpha, or a graph load.
Sizes are those of the repository's own workloads (10k nodes / 50k edges up to
50M nodes / 500M edges) and ragged ones between them.

A program keeps one context with its graph loaded and sends it queries, so the
context of a graph is kept here as well (the handle), made from the case's
sizes alone; what the seed decides are the queries (for a graph load, the
graph; for a new alpha, alpha and the query).  Graphs follow the repository's
generator: Chung-Lu power-law degrees for sources and a permuted copy for
targets, uniform labels, reverse edges, 1-3 Zipf keywords per node, optional
hubs; they are built on the GPU since they are made many times.
"""
from __future__ import annotations

import collections
import math

import numpy as np
import torch

import paper_2001_06770_amd as raks

# Common settings: power-law exponent, labels, Zipf exponent and the number of
# frequent keywords that queries draw from are the generator's own.
BASE = {"pl": 2.1, "labels": 100, "hubs": False, "abar": 3.05, "node_mode": False,
        "score_mode": 0, "rerank": 0, "queries": 1, "limit": 20}
ZIPF, TOP = 1.1, 200


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the smallest call: one query on a graph of the small workload's size;
        # launches and host round trips are all there is
        _case("one_small", kind="query", nodes=10_000, edges=50_000, vocab=2000, abar=3.03,
              c_lo=2, c_hi=2, m_lo=2, m_hi=2, k=10, w=10),
        # a tight serving loop that may not allocate: ragged middle-sized graph
        _case("noalloc_ragged", kind="noalloc", nodes=300_007, edges=2_345_679, vocab=20_011,
              c_lo=2, c_hi=3, m_lo=1, m_hi=2, k=10, w=16),
        # the ordinary interactive query (medium workload)
        _case("one_medium", kind="query", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=3, c_hi=3, m_lo=3, m_hi=3, k=20, w=20),
        # many keywords (rows of 16 and 8 levels), product score, re-ranked ties
        _case("wide_rerank", kind="query", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=9, c_hi=11, m_lo=5, m_hi=8, k=20, w=40, score_mode=1, rerank=1),
        # no marginal keywords, levels from node weights, ragged sizes
        _case("central_node_mode", kind="query", nodes=777_777, edges=5_555_555, vocab=31_337,
              abar=3.2, node_mode=True, c_lo=3, c_hi=5, m_lo=0, m_hi=0, k=20, w=20),
        # a user turning the granularity knob: new alpha, then the same kind of query
        _case("new_alpha", kind="alpha", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=3, c_hi=3, m_lo=3, m_hi=3, k=20, w=20),
        # a graph (re)load, as a service does when its data changes, with its levels read back
        _case("load_graph", kind="load", nodes=1_500_003, edges=12_345_678, vocab=50_021,
              abar=3.1),
        # offline batch of 32 queries sharing level loops (medium workload)
        _case("batch_medium", kind="batch", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=3, c_hi=3, m_lo=3, m_hi=3, k=20, w=20, queries=32),
        # the same kind of batch over independent lanes
        _case("lanes_medium", kind="lanes", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=2, c_hi=4, m_lo=2, m_hi=4, k=20, w=20, queries=32),
        # served queries: 24 arrive together at a running server
        _case("served_medium", kind="serve", nodes=2_000_000, edges=20_000_000, vocab=100_000,
              c_lo=2, c_hi=5, m_lo=2, m_hi=5, k=20, w=20, queries=24),
        # one query of many keywords on a large graph with planted hubs (large workload)
        _case("one_large_hubs", kind="query", nodes=20_000_000, edges=200_000_000, vocab=1_000_000,
              pl=2.0, hubs=True, abar=3.47, c_lo=5, c_hi=5, m_lo=5, m_hi=5, k=50, w=50, limit=12),
        # the largest: a batch of mixed queries on the serving graph
        _case("batch_serving_graph", kind="batch", nodes=50_000_000, edges=500_000_000,
              vocab=1_000_000, abar=3.29, c_lo=2, c_hi=5, m_lo=2, m_hi=5, k=20, w=20, queries=12),
    ]


def draw(rng):
    """A case of the listed ranges: kind, graph size, keyword counts, beam and options."""
    kind = rng.choice(["query"] * 4 + ["batch"] * 3 + ["lanes", "serve", "noalloc", "alpha", "load"])
    top = {"query": 20e6, "batch": 4e6, "lanes": 4e6, "serve": 4e6, "noalloc": 3e5, "alpha": 4e6,
           "load": 2e6}[kind]
    n = int(math.exp(rng.uniform(math.log(10_000), math.log(top))))
    ratio = rng.uniform(5.0, 10.0)
    c, m = rng.randint(1, 6), rng.choice([0, 1, 2, 3, 4, 6])
    if c + m < 3:   # one central + one marginal keyword can recover most of a graph
        c, m = 2, 1
    k = rng.choice([5, 10, 20, 50])
    if kind == "noalloc":   # its scratch bounds nodes and beam
        k, c, m = min(k, 20), min(c, 4), min(m, 3)
    several = kind in ("batch", "lanes", "serve")
    return _case("", kind=kind, nodes=n, edges=int(n * ratio), vocab=max(2000, n // 20),
                 abar=round(3.4 - 0.07 * (ratio - 5.0), 2), node_mode=rng.random() < 0.25,
                 c_lo=c, c_hi=min(c + rng.randint(0, 2), 8), m_lo=m, m_hi=m, k=k,
                 w=k + rng.choice([0, 0, 7, k] if kind != "noalloc" else [0]), score_mode=int(rng.random() < 0.2),
                 rerank=int(rng.random() < 0.2), queries=rng.randint(3, 40) if several else 1)


# ------------------------------------------------------------------ graphs


class Graph:
    """Host arrays of a bi-directed CSR graph, rows sorted by (label, destination)."""


def _power_law(n, pl, gen):
    u = 1.0 - torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    return torch.clamp(torch.floor(u ** (-1.0 / (pl - 1.0))), 1, n - 1).to(torch.int64)


def _sample(cum, count, gen):
    """``count`` indices drawn in proportion to integer weights (their running sums)."""
    r = torch.randint(0, int(cum[-1]), (count,), generator=gen, device="cuda")
    return torch.searchsorted(cum, r, right=True)


def _distinct(keys):
    keys = torch.sort(keys)[0]
    keep = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
    keep[1:] = keys[1:] != keys[:-1]
    return keys[keep]


def make_graph(case, seed):
    n, edges, labels, vocab = case["nodes"], case["edges"], case["labels"], case["vocab"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    weight = _power_law(n, case["pl"], gen)
    cum_out = torch.cumsum(weight, 0)
    cum_in = torch.cumsum(weight[torch.randperm(n, generator=gen, device="cuda")], 0)
    # exactly `edges` distinct undirected (node, label, node) triples: some more
    # than needed, without self-loops and duplicates, the surplus left out evenly
    more = 1.06
    while True:
        cnt = int(edges * more) + 64
        src = _sample(cum_out, cnt, gen)
        if case["hubs"]:   # four nodes with 0.5 to 1 % of all edges each
            at = 0
            for i, share in enumerate((200, 167, 133, 100)):
                src[at:at + edges // share] = (n // 5) * (i + 1) - 1
                at += edges // share
        dst = _sample(cum_in, cnt, gen)
        lab = torch.randint(0, labels, (cnt,), generator=gen, device="cuda")
        keep = src != dst
        keys = ((torch.minimum(src, dst) * labels + lab) * n + torch.maximum(src, dst))[keep]
        in_deg = torch.bincount(dst, minlength=n)
        del src, dst, lab, keep
        keys = _distinct(keys)
        if keys.numel() >= edges:
            break
        more *= 1.25
    pick = torch.arange(edges, device="cuda") * keys.numel() // edges
    keys = keys[pick]
    hi = keys % n
    keys //= n
    lab = keys % labels
    keys //= labels
    arcs = torch.cat([(keys * labels + lab) * n + hi, (hi * labels + lab) * n + keys])
    del keys, hi, lab, pick, weight, cum_out, cum_in
    arcs = torch.sort(arcs)[0]
    g = Graph()
    g.n_nodes, g.abar = n, case["abar"]
    g.col = (arcs % n).to(torch.int32).cpu().numpy()
    arcs //= n
    g.label = (arcs % labels).to(torch.int16).cpu().numpy().view(np.uint16)
    arcs //= labels
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(arcs, minlength=n), 0)
    g.row_ptr = row_ptr.cpu().numpy()
    del arcs, row_ptr
    g.node_weight = torch.clamp(torch.floor(8 * torch.log2(1 + in_deg.double()) + 0.5), max=255
                                ).to(torch.uint8).cpu().numpy()
    # 1-3 keywords per node from a truncated Zipf law
    zipf = (1e9 / torch.arange(1, vocab + 1, device="cuda", dtype=torch.float64) ** ZIPF).long() + 1
    cum = torch.cumsum(zipf, 0)
    cnt = torch.randint(1, 4, (n,), generator=gen, device="cuda")
    node = torch.repeat_interleave(torch.arange(n, device="cuda"), cnt)
    pairs = _distinct(_sample(cum, node.numel(), gen) * n + node)
    g.kw_nodes = (pairs % n).to(torch.int32).cpu().numpy()
    kw_ptr = torch.zeros(vocab + 1, dtype=torch.int64, device="cuda")
    kw_ptr[1:] = torch.cumsum(torch.bincount(pairs // n, minlength=vocab), 0)
    g.kw_ptr = kw_ptr.cpu().numpy()
    del pairs, node, cnt, cum, zipf, kw_ptr, in_deg
    torch.cuda.empty_cache()
    return g


# ------------------------------------------------------------------ handles

Query = collections.namedtuple("Query", "central marginal k w max_level score_mode rerank")
GRAPH_KEYS = ("nodes", "edges", "pl", "labels", "vocab", "hubs", "abar", "node_mode")
KEEP_BYTES = 100 << 30
_handles = collections.OrderedDict()


class Handle:
    """A context with its graph loaded, and the graph's most frequent keywords."""

    def __init__(self, case):
        g = make_graph(case, 1)
        kind = case["kind"]
        self.ctx = raks.Context(0, lanes=4 if kind == "lanes" else 1)
        self.ctx.load_graph(g, alpha=0.5, mode=int(case["node_mode"]))
        if kind == "lanes":
            self.ctx.set_batch_mode(raks.RAKS_BATCH_LANES)
        if kind == "serve":
            self.ctx.serve_start()
        freq = np.diff(g.kw_ptr)
        self.top = np.argsort(-freq, kind="stable")[:TOP]
        self.bytes = int(g.col.shape[0]) * 24 + case["nodes"] * 400


def _handle(case):
    own = case["kind"] if case["kind"] in ("lanes", "serve", "alpha") else "plain"
    key = (own,) + tuple(case[k] for k in GRAPH_KEYS)
    if key not in _handles:
        while _handles and sum(h.bytes for h in _handles.values()) > KEEP_BYTES:
            _handles.popitem(last=False)
        _handles[key] = Handle(case)
    _handles.move_to_end(key)
    return _handles[key]


def _queries(case, top, rng):
    out = []
    for _ in range(case["queries"]):
        nc = int(rng.integers(case["c_lo"], case["c_hi"] + 1))
        nm = int(rng.integers(case["m_lo"], case["m_hi"] + 1))
        pick = [int(x) for x in rng.choice(top, size=nc + nm, replace=False)]
        out.append(Query(tuple(pick[:nc]), tuple(pick[nc:]), case["k"], case["w"], case["limit"],
                         case["score_mode"], case["rerank"]))
    return out


def prepare(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    state = {"kind": case["kind"]}
    if case["kind"] == "load":
        state["graph"] = make_graph(case, 1000 + seed)
        state["mode"] = int(case["node_mode"])
        key = ("load",)
        if key not in _handles:
            _handles[key] = collections.namedtuple("Loader", "ctx bytes")(raks.Context(0), 1 << 30)
        state["ctx"] = _handles[key].ctx
        return state
    h = _handle(case)
    state["ctx"] = h.ctx
    state["queries"] = _queries(case, h.top, rng)
    state["buffers"] = Buffers(case)
    state["alpha"] = round(float(rng.uniform(0.2, 0.8)), 3)
    return state


# ------------------------------------------------------------------ a pass


class Buffers:
    """A client's result buffers: per query its status and counters, per result
    its scores and list sizes, and all lists back to back (what does not fit is
    left out; the sizes tell).  They hold the last pass."""

    def __init__(self, case):
        nq, several = case["queries"], case["queries"] > 1
        self.k = case["k"]
        self.stats = np.zeros((nq, 17), np.int64)
        self.meta = np.full((nq, self.k, 7), -1, np.int64)
        self.nodes = np.zeros(1 << (22 if several else 18), np.int32)
        self.arcs = np.zeros((1 << (22 if several else 19), 3), np.int32)

    def take(self, rs):
        at_n = at_a = 0
        for i, r in enumerate(rs):
            row = [r["status"], r["n_cg"], len(r["results"])]
            for st in r["stats"]:
                row += [st["levels"], st["end_reason"], st["frontier"], st["e_arc"], st["e_alg"],
                        st["gate_pass"], st["h_writes"]]
            self.stats[i] = row
            meta = []
            for x in r["results"]:
                nodes, arcs = x["nodes"], x["arcs"]
                nn, na = len(nodes), len(arcs)
                meta.append((x["central"], x["score_c"], x["score_m"], x["key"], x["weight_sum"],
                             nn, na))
                if at_n + nn <= len(self.nodes):
                    self.nodes[at_n:at_n + nn] = nodes
                    at_n += nn
                if at_a + na <= len(self.arcs):
                    self.arcs[at_a:at_a + na] = arcs
                    at_a += na
            if meta:
                self.meta[i, :len(meta)] = meta
        return {"stats": self.stats, "meta": self.meta, "nodes": self.nodes, "arcs": self.arcs}


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "load":
        ctx.load_graph(state["graph"], alpha=0.5, mode=state["mode"])
        return ctx.activations()
    qs, take = state["queries"], state["buffers"].take
    if kind == "query":
        return take([ctx.query(qs[0], lean=True)])
    if kind == "noalloc":
        return take([ctx.query_noalloc(qs[0], lean=True)])
    if kind == "alpha":
        ctx.set_alpha(state["alpha"])
        return take([ctx.query(qs[0], lean=True)])
    if kind == "serve":
        tickets = [ctx.submit(q) for q in qs]
        return take([ctx.wait(t, lean=True) for t in tickets])
    return take(ctx.query_batch(qs, lean=True))   # batch (cohorts) and lanes


def work(case):
    """Bytes one pass cannot do without: per run the keyword matrix written
    once, and the id and level (5 bytes) of the arcs that a run of these
    queries reads before its stop rule, about 0.4 of all arcs; a batch reads
    an arc once for all its queries.  A load reads its arrays once and writes
    levels and the level-ordered arcs once; a new alpha reads label counts and
    arcs and writes levels and ordered arcs."""
    n, arcs = case["nodes"], 2 * case["edges"]
    if case["kind"] == "load":
        return {"bytes": 6.0 * arcs + 17.0 * n + 5.0 * arcs + 1.0 * arcs, "flops": 0.0}
    cols = (case["c_lo"] + case["c_hi"] + case["m_lo"] + case["m_hi"]) / 2.0
    runs = 2 if case["m_hi"] else 1
    b = 0.4 * runs * 5.0 * arcs + case["queries"] * cols * n
    if case["kind"] == "alpha":
        b += (4.0 + 4.0 + 1.0 + 5.0) * arcs
    return {"bytes": b, "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number, equal on every correct path."""
    return None
