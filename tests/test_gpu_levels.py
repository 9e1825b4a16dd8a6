"""Traversal copy (rows ordered by activation level) at the edges of its row
size classes: hubs whose degrees sit around the group, wavefront and tile
sizes, in both activation modes and with more levels than the level table
holds.  The activation levels, every result and every work counter equal the
reference implementation's."""
from __future__ import annotations

import numpy as np
import pytest

import graphs
import oracle
import synth

pytestmark = pytest.mark.gpu

DEGREES = (1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 4095,
           255, 256, 257, 4096, 4097, 8193, 9001, 16384, 16385, 17000)


def hub_graph(seed, more):
    """One hub per degree (and `more` of 65 to 300 arcs), its edges going to a
    shared pool of leaves and to the other hubs' leaves; labels of very different
    counts."""
    rng = np.random.default_rng(seed)
    degrees = DEGREES + tuple(int(x) for x in rng.integers(65, 301, size=more))
    hubs, leaves = len(degrees), 18_000
    n = hubs + leaves + 7   # some isolated nodes
    edges = set()
    for h, d in enumerate(degrees):
        for v in rng.choice(leaves, size=d, replace=False):
            edges.add((h, hubs + int(v), int(min(rng.geometric(0.3), 12))))
    keywords = [sorted(set(int(x) for x in rng.integers(0, n, size=k))) for k in (3, 5, 9, 40, 200, 2)]
    weight = rng.integers(0, 200, size=n).astype(np.uint8)
    return graphs.build(n, edges, keywords, node_weight=weight)


@pytest.mark.parametrize("abar_x100", [305, 4000])
@pytest.mark.parametrize("mode", [0, 1], ids=["edge", "node"])
@pytest.mark.parametrize("more", [0, 700])   # all middle classes in one launch, one launch each
def test_row_size_classes(more, mode, abar_x100):
    import paper_2001_06770_amd as raks
    g = hub_graph(abar_x100 + mode, more)
    g.abar_x100 = abar_x100
    o = oracle.Oracle(g)
    with raks.Context(0, poison=0xA5) as ctx:
        ctx.load_graph(g, alpha=0.4, mode=mode)
        for alpha in (0.4, 0.7):
            if alpha != 0.4:
                ctx.set_alpha(alpha)
            act = o.activation(g.abar, alpha, mode)
            act = act[0] if mode else act
            np.testing.assert_array_equal(ctx.activations(), act)
            for q in (synth.Query((0, 1), (2, 3), 5, 9, 60), synth.Query((4, 5), (), 7, 7, 60),
                      synth.Query((3,), (4, 0, 1), 4, 20, 60)):
                got = ctx.query(q)
                for key in ("device_ms", "host_ms", "queue_ms"):
                    got.pop(key)
                assert got == o.query(act, q), (alpha, q)


@pytest.mark.parametrize("drop", ["hub_to_leaf", "leaf_to_hub", "leaf_to_leaf", "both_sides"])
def test_missing_reverse_arc_rejected(drop):
    """A graph with one arc's reverse taken out breaks the contract, whichever
    end has the larger row; so does one that lacks as many arcs on either side."""
    import paper_2001_06770_amd as raks
    g = graphs.build(1200, [(0, v, v % 3) for v in range(1, 1101)] + [(1150, 1151, 2), (1, 2, 0)],
                     [[0], [1]])

    def without(src, dst):
        e = int(g.row_ptr[src]) + int(np.nonzero(g.col[g.row_ptr[src]:g.row_ptr[src + 1]] == dst)[0][0])
        g.col, g.label = np.delete(g.col, e), np.delete(g.label, e)
        g.row_ptr = g.row_ptr - (np.arange(g.row_ptr.shape[0]) > src)

    with raks.Context(0) as ctx:
        ctx.load_graph(g, alpha=0.5)
        if drop in ("hub_to_leaf", "both_sides"):
            without(0, 700)
        if drop in ("leaf_to_hub", "both_sides"):
            without(801, 0)
        if drop == "leaf_to_leaf":
            without(1151, 1150)
        with pytest.raises(raks.RaksError) as e:
            ctx.load_graph(g, alpha=0.5)
        assert e.value.code == -1
