"""raks_query_noalloc: the scratch beside the node buffers belongs to the recovered
lists, and graphs are refused by their size alone."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from test_gpu_long_lists import fan
from test_zz_no_alloc import chain

pytestmark = pytest.mark.gpu


def test_recovered_lists_get_the_scratch():
    """A graph of 2.9M nodes whose result of 140k nodes needs about 100 MB of lists."""
    import paper_2001_06770_amd as raks
    g = fan(140_000, 2_800_000)
    q = synth.Query((0,), (1,), 1, 1)
    with raks.Context(0) as ctx:
        ctx.load_graph(g, alpha=0.5)
        got, exp = ctx.query_noalloc(q, lean=True), ctx.query(q, lean=True)
    assert got["stats"] == exp["stats"] and len(got["results"]) == len(exp["results"]) == 1
    for a, b in zip(got["results"], exp["results"]):
        assert len(a["nodes"]) == 140_002
        for key in a:
            np.testing.assert_array_equal(a[key], b[key])


@pytest.mark.parametrize("n,fits", [(4_500_000, True), (4_650_000, False)])
def test_graphs_are_taken_by_their_nodes(n, fits):
    """50 bytes and two rows of four hitting levels per node, in 256 MiB."""
    import paper_2001_06770_amd as raks
    padded = -(-n // 1024) * 1024
    assert (padded * 58 <= 256 << 20) == fits
    g = chain(n)
    q = synth.Query((0,), (1,), 1, 1)
    with raks.Context(0) as ctx:
        ctx.load_graph(g, alpha=0.5)
        if fits:
            got, exp = ctx.query_noalloc(q), ctx.query(q)
            assert got["stats"] == exp["stats"] and got["results"] == exp["results"]
        else:
            with pytest.raises(raks.RaksError) as e:
                ctx.query_noalloc(q)
            assert e.value.code == -2 and "4650000 nodes" in str(e.value)
