"""Result lists around the sizes where the union of a result's lists changes its
way (counting, LDS radix sort, id slices over many workgroups), for central
graphs and for results, with and without marginal keywords, re-ranked and not,
on graphs of one and of several id slices."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu


def fan(width, tail=0):
    """Keyword 0 on node 0, keyword 1 on node 1, `width` middle nodes between
    them: a result holds all middle nodes and their arcs.  `tail` further nodes
    with arcs among themselves only widen the id range."""
    n = 3 + width + tail
    mids = np.arange(3, 3 + width)
    t = np.arange(3 + width, n)
    src = np.concatenate([np.zeros(width, np.int64), np.ones(width, np.int64), [2], t[:-1]])
    dst = np.concatenate([mids, mids, [0], t[1:]])
    s, d = np.concatenate([src, dst]), np.concatenate([dst, src])
    perm = np.random.default_rng(width + tail).permutation(n)   # ids in no order
    s, d = perm[s], perm[d]
    order = np.lexsort((d, s))
    s, d = s[order], d[order]
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(s, minlength=n))
    kw = [[int(perm[0])], [int(perm[1])], [int(perm[2])], sorted(int(perm[x]) for x in mids[:50])]
    return graphs.G(n, row_ptr, d.astype(np.int32), np.zeros(d.shape[0], np.uint16),
                    np.zeros(n, np.uint8), np.cumsum([0] + [len(k) for k in kw]).astype(np.int64),
                    np.concatenate(kw).astype(np.int32))


def run(ctx, o, act, queries):
    for q in queries:
        exp = o.query(act, q)
        for got in (ctx.query(q), ctx.query_batch([q, q])[1]):
            for key in ("device_ms", "host_ms", "queue_ms"):
                got.pop(key)
            assert got == exp, q


@pytest.mark.parametrize("width", [120, 255, 256, 511, 512, 513, 2046, 2049, 4095, 4096, 4097, 9000])
def test_list_lengths(width):
    import paper_2001_06770_amd as raks
    g = fan(width)
    o = oracle.Oracle(g)
    act = o.activation(g.abar, 0.5)
    with raks.Context(0, poison=0xA5) as ctx:
        ctx.load_graph(g, alpha=0.5)
        run(ctx, o, act, [synth.Query((0,), (1,), 2, 3), synth.Query((0, 1), (), 3, 3),
                          synth.Query((1,), (2, 3), 1, 2), synth.Query((3,), (0, 1), 4, 9, rerank=1),
                          synth.Query((2,), (1,), 1, 1, rerank=1)])


@pytest.mark.parametrize("width,tail", [(5000, 1 << 20), (20_000, 600_000)])
def test_several_id_slices(width, tail):
    import paper_2001_06770_amd as raks
    g = fan(width, tail)
    o = oracle.Oracle(g, check=False)
    act = o.activation(g.abar, 0.5)
    with raks.Context(0, poison=0x5A) as ctx:
        ctx.load_graph(g, alpha=0.5)
        run(ctx, o, act, [synth.Query((0,), (1,), 2, 2), synth.Query((0, 1), (), 2, 2),
                          synth.Query((1,), (2, 3), 1, 4, rerank=1)])


def test_small_graph_floods():
    """Queries of one or two keywords recover most of the graph."""
    import paper_2001_06770_amd as raks
    g = synth.make_graph("small")
    o = oracle.Oracle(g)
    act = o.activation(g.abar, 0.5)
    top = [int(x) for x in synth.top_keywords(g, 200)]
    qs = [synth.Query((top[-1 - i],), tuple(top[150 - 3 * i - j] for j in range(1 + i % 2)), 10, 20,
                      rerank=i % 3 == 0) for i in range(12)]
    with raks.Context(0, poison=0xFF, big_list=30_000) as ctx:
        ctx.load_graph(g, alpha=0.5)
        run(ctx, o, act, qs)
