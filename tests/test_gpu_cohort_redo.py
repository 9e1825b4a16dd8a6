"""Cohort batches whose central-graph stages run out of their capacities and are
repeated while nothing else runs: the level loop waits for the repeats, whenever
it sees the first attempt end."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu


def hub_graph():
    """Three hubs with half of the arcs of 1025 nodes, frequent keywords."""
    rng = np.random.default_rng(36)
    n, e = 1025, 2000
    hubs = rng.integers(0, n, 3)
    src = np.where(rng.random(e) < 0.4, rng.choice(hubs, e), rng.integers(0, n, e))
    edges = zip(src.tolist(), rng.integers(0, n, e).tolist(), rng.integers(0, 2, e).tolist())
    kws = [np.unique(rng.integers(0, n, c)).tolist() for c in (3, 20, 200, 60, 5, 100, 2, 30)]
    return graphs.build(n, edges, kws, abar_x100=1000)


def test_repeated_stages_are_waited_for():
    """Nothing is left to explore beside the stages of queries without marginal
    keywords; queries of their own alpha run on other lanes and the first batch of a
    context makes its lanes, so the loop often looks at a stage just as it ends."""
    import paper_2001_06770_amd as raks
    g = hub_graph()
    o = oracle.Oracle(g)
    act = {0.0: o.activation(g.abar, 0.5), 0.3: o.activation(g.abar, 0.3)}
    shared = [synth.Query((1, 3, 4), (), 20, 64, 60), synth.Query((3, 7, 2), (), 2, 5, 125),
              synth.Query(tuple(range(8)), (), 20, 256, 60)]
    single = [synth.Query((0, 2, 5), (6, 1, 7), 20, 256, 60, alpha=0.3),
              synth.Query((3, 1), (5,), 20, 64, 60, alpha=0.3, rerank=1),
              synth.Query((2, 4), (6, 0), 5, 64, 60, alpha=0.3)]
    exp = {q: o.query(act[q.alpha], q) for q in shared + single}
    for i in range(60):
        qs = single + [shared[i % 3]] + single + single[:2]
        with raks.Context(0, lanes=3, rec_caps=(1, 1, 1), poison=0x68) as ctx:
            ctx.load_graph(g, alpha=0.5)
            for q, got in zip(qs, ctx.query_batch(qs)):
                for key in ("device_ms", "host_ms", "queue_ms"):
                    got.pop(key)
                assert got == exp[q], (i, q)
