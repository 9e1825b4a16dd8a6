"""Queries whose columns start and end anywhere in a segment of the cohort, with
copies of 4, 8 and 16 bytes per node: the copy, the counters and the reset of a
query's columns touch exactly its own bytes, whatever its neighbours in the row
still do.  Every result and counter equals the oracle's."""
from __future__ import annotations

import random

import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("totals", [(1, 2, 3, 4), (5, 8, 3), (9, 7), (15, 1), (16,), (2, 13, 1, 6)])
def test_columns_anywhere_in_a_segment(totals):
    import paper_2001_06770_amd as raks
    g = synth.make_graph("tiny2")
    o = oracle.Oracle(g)
    act = o.activation(g.abar, 0.5)
    rnd = random.Random(sum(totals))
    pool = [int(x) for x in synth.top_keywords(g, 100)]
    qs = []
    for i in range(24):
        t = totals[i % len(totals)]
        c = rnd.randint(max(1, t - 8), min(t, 8))
        kws = rnd.sample(pool, t)
        k = rnd.randint(1, 9)
        qs.append(synth.Query(tuple(kws[:c]), tuple(kws[c:]), k, k + rnd.randint(0, 6),
                              max_level=rnd.choice([1, 2, 3, 20])))
    exp = [o.query(act, q) for q in qs]
    with raks.Context(0, poison=0x5A) as ctx:
        ctx.load_graph(g, alpha=0.5)
        for rep in range(2):   # a second batch finds every byte reset
            for q, got, e in zip(qs, ctx.query_batch(qs), exp):
                for key in ("device_ms", "host_ms", "queue_ms"):
                    got.pop(key)
                assert got == e, (rep, q)
