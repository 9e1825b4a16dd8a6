"""Top-w selection over many workgroups, the levels' staged central nodes and the
expansion's tiles at the edges of their ranges: graphs whose central nodes all
tie, lie in one scan workgroup or are spread over all of them, with beams at
the limits, and rows whose slices end at tile borders."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu


def check(g, queries, alpha=0.5):
    import paper_2001_06770_amd as raks
    o = oracle.Oracle(g)
    act = o.activation(g.abar, alpha)
    with raks.Context(0, poison=0x5A) as ctx:
        ctx.load_graph(g, alpha=alpha)
        for q in queries:
            exp = o.query(act, q)
            for got in (ctx.query(q), ctx.query_batch([q])[0]):
                for key in ("device_ms", "host_ms", "queue_ms"):
                    got.pop(key)
                assert got == exp, q


@pytest.mark.parametrize("leaves", [255, 1024, 4096, 4097, 33 * 1024 + 5, 70_001])
def test_many_tied_central_nodes(leaves):
    """Every leaf of two hubs is a central node of the two hub keywords: one
    level's candidates, all with the same sum, spread over all scan workgroups
    (the leaves have equal rows); ties go to the smallest ids."""
    n = leaves + 2
    src = np.repeat([0, 1], leaves)
    dst = np.tile(np.arange(2, n), 2)
    s, d = np.concatenate([src, dst]), np.concatenate([dst, src])
    order = np.lexsort((d, s))
    s, d = s[order], d[order]
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(s, minlength=n))
    kw = [[0], [1], [2, n - 1], [n // 2]]
    g = graphs.G(n, row_ptr, d.astype(np.int32), np.zeros(d.shape[0], np.uint16),
                 np.zeros(n, np.uint8), np.cumsum([0] + [len(k) for k in kw]).astype(np.int64),
                 np.concatenate(kw).astype(np.int32))
    check(g, [synth.Query((0, 1), (), 1, 1), synth.Query((0, 1), (2,), 3, 17),
              synth.Query((0, 1), (2, 3), 250, 256), synth.Query((1, 3), (0,), 5, 200)])


@pytest.mark.parametrize("row", [1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1025])
def test_rows_at_tile_borders(row):
    """A chain of hubs with `row` leaves each: their slices fill tiles exactly,
    or end one arc before or after, and a tile holds up to 256 one-arc entries."""
    rng = np.random.default_rng(row)
    hubs, edges = 9, set()
    n = hubs * (row + 1)
    for h in range(hubs):
        for i in range(row):
            edges.add((h, hubs + h * row + i, int(rng.integers(0, 4))))
        if h:
            edges.add((h - 1, h, 1))
    kws = [[0], [hubs - 1], [hubs], [n - 1], sorted(set(int(x) for x in rng.integers(0, n, 300)))]
    g = graphs.build(n, edges, kws)
    check(g, [synth.Query((0, 1), (2, 3), 4, 8), synth.Query((0,), (1, 4), 9, 30),
              synth.Query((2, 3, 4), (), 3, 3), synth.Query((4,), (0, 1, 2, 3), 6, 40)])
