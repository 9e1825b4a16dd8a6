"""The RPG check over many central-keyword nodes: V_C sizes around the ones where
the check spreads over more workgroups, one and several central graphs, nodes that
several keywords' searches reach, short and long recovered lists (per-instance node
sets, bitmaps, labels).  Results and work counters, whose levels tell when every RPG
was found, equal the reference implementation's."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu


def spokes(hubs, n_spokes, k, chain=5):
    """`hubs` nodes, each joined to the first node of every spoke; a spoke has k nodes
    that carry keywords 0..k-1 (even spokes) or k..2k-1 (odd ones), so only hubs see all
    of them.  Chains of `chain` and `chain` + 3 nodes lead from spoke ends to keywords
    2k and 2k + 1; keyword 2k + 2 is on every tenth spoke's end."""
    first = hubs + k * np.arange(n_spokes)
    edges = [(h, int(f), 0) for h in range(hubs) for f in first]
    edges += [(int(f) + i, int(f) + i + 1, 0) for f in first for i in range(k - 1)]
    kw = [[] for _ in range(2 * k + 3)]
    for i in range(k):
        kw[i] = [int(f) + i for f in first[::2]]
        kw[k + i] = [int(f) + i for f in first[1::2]]
    n = hubs + k * n_spokes
    for c in range(2):
        at = int(first[c]) + k - 1
        for _ in range(chain + 3 * c):
            edges.append((at, n, 1 + c))
            at, n = n, n + 1
        kw[2 * k + c] = [at]
    kw[2 * k + 2] = [int(f) + k - 1 for f in first[::10]]
    perm = np.random.default_rng(n).permutation(n)   # ids in no order
    return graphs.build(n, [(int(perm[u]), int(perm[v]), lab) for u, v, lab in edges],
                        [[int(perm[x]) for x in nodes] for nodes in kw])


@pytest.mark.parametrize("hubs,n_spokes,k", [(1, 4095, 1), (1, 4096, 1), (1, 4097, 1), (2, 4100, 1),
                                             (3, 2731, 1), (1, 2400, 3), (2, 9001, 2), (1, 9000, 8)])
@pytest.mark.parametrize("rec_caps", [(0, 0, 0), (64, 64, 64)], ids=["default", "small_caps"])
def test_many_central_keyword_nodes(hubs, n_spokes, k, rec_caps):
    import paper_2001_06770_amd as raks
    g = spokes(hubs, n_spokes, k)
    o = oracle.Oracle(g)
    act = o.activation(g.abar, 0.5)
    central = tuple(range(2 * k))
    qs = [synth.Query(central, (2 * k, 2 * k + 1), hubs, hubs, 60),
          synth.Query(central[:-1], (2 * k + 1,), 1, 2, 60, rerank=1)]
    if k < 8:
        qs.append(synth.Query(central, (2 * k, 2 * k + 2), 1, 3, 60, score_mode=1))
    with raks.Context(0, poison=0x5A, rec_caps=rec_caps) as ctx:
        ctx.load_graph(g, alpha=0.5)
        for q in qs:
            exp = o.query(act, q)
            if q is qs[0]:
                assert len(exp["results"]) == hubs
                vc = len({x for t in central for x in graphs.keyword_nodes(g, t)})
                assert vc == n_spokes * k and exp["stats"][1]["levels"] > 5
            for got in (ctx.query(q), ctx.query_batch([q, q])[1]):
                for key in ("device_ms", "host_ms", "queue_ms"):
                    got.pop(key)
                assert got == exp, q
