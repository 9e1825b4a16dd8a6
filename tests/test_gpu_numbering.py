"""The degree order of the nodes at the edges of the numbering's tiles (4096 ids,
1024 per wavefront) and digits (degrees around 255, 256 and 65536), with equal
degrees and nodes without arcs: every answer comes back in original ids, so a wrong
or repeated internal number shows in any of them."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hubs", [(1, ()), (2, (1,)), (1023, (255,)), (1024, (256, 257)),
                                    (1025, (255, 256, 1)), (4095, (300, 300, 2)),
                                    (4096, (4000, 255, 255)), (4097, (257,)), (9000, (8192, 511, 512)),
                                    (70_000, (65_535, 65_536, 65_537, 256))])
def test_degree_order(n, hubs):
    import paper_2001_06770_amd as raks
    rng = np.random.default_rng(n)
    edges = set()
    for h, d in enumerate(hubs):
        # hubs spread over the ids, the last one the last id
        hub = n - 1 - h * (n // (2 * len(hubs) + 1))
        pool = np.delete(np.arange(n), hub)
        for v in rng.choice(pool, size=d, replace=False):
            edges.add((hub, int(v), int(v) % 3))
    kws = [sorted(set(int(x) for x in rng.integers(0, n, size=k))) for k in (1, 2, 5, 30)]
    g = graphs.build(n, edges, kws)
    o = oracle.Oracle(g)
    act = o.activation(g.abar, 0.5)
    with raks.Context(0, poison=0xA5) as ctx:
        ctx.load_graph(g, alpha=0.5)
        np.testing.assert_array_equal(ctx.activations(), act)
        for q in (synth.Query((0, 1), (2,), 3, 5), synth.Query((3,), (0, 1, 2), 10, 20),
                  synth.Query((2, 3), (), 6, 6)):
            got = ctx.query(q)
            for key in ("device_ms", "host_ms", "queue_ms"):
                got.pop(key)
            assert got == o.query(act, q), q
