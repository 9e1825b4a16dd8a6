"""Graphs that break the input contract in several ways at once: the error names
every kind of violation, as a check of each arc by itself finds them."""
from __future__ import annotations

import re

import numpy as np
import pytest

import graphs

pytestmark = pytest.mark.gpu


def violations(g):
    """1 col range, 2 self-loop, 4 row order, 8 missing reverse arc, arc by arc."""
    key = list(zip(g.label.tolist(), g.col.tolist()))
    bits = 0
    for u in range(g.n_nodes):
        for e in range(int(g.row_ptr[u]), int(g.row_ptr[u + 1])):
            lab, v = key[e]
            if not 0 <= v < g.n_nodes:
                bits |= 1
                continue
            bits |= 2 * (u == v) | 4 * (e > g.row_ptr[u] and key[e - 1] >= key[e])
            a, b = int(g.row_ptr[v]), int(g.row_ptr[v + 1])
            hi = b
            while a < b:
                m = (a + b) // 2
                if key[m] < (lab, u):
                    a = m + 1
                else:
                    b = m
            bits |= 8 * (a == hi or key[a] != (lab, u))
    return bits


def insert(g, u, at, lab, v):
    e = int(g.row_ptr[u]) + at
    g.label, g.col = np.insert(g.label, e, lab), np.insert(g.col, e, v)
    g.row_ptr = g.row_ptr + (np.arange(g.row_ptr.shape[0]) > u)


def delete(g, u, v):
    e = int(g.row_ptr[u]) + int(np.nonzero(g.col[g.row_ptr[u]:g.row_ptr[u + 1]] == v)[0][0])
    g.label, g.col = np.delete(g.label, e), np.delete(g.col, e)
    g.row_ptr = g.row_ptr - (np.arange(g.row_ptr.shape[0]) > u)


CASES = {
    "loop_and_hub_side": (0xA, [("del", 0, 700), ("ins", 5, 1, 9, 5)]),
    "loop_and_leaf_side": (0xA, [("del", 700, 0), ("ins", 5, 1, 9, 5)]),
    "loop_alone": (0x2, [("ins", 5, 1, 9, 5)]),
    "range_and_hub_side": (0x9, [("del", 0, 700), ("ins", 5, 1, 9, 4000)]),
    "loop_out_of_order": (0xE, [("ins", 4, 1, 0, 4)]),
    "all": (0xF, [("del", 0, 700), ("ins", 5, 1, 9, -1), ("ins", 4, 1, 0, 4)]),
    "hub_side_alone": (0x8, [("del", 0, 700)]),
}


@pytest.mark.parametrize("name", CASES)
def test_every_violation_is_named(name):
    import paper_2001_06770_amd as raks
    g = graphs.build(1200, [(0, v, v % 3) for v in range(1, 1101)], [[0], [1]])
    bits, edits = CASES[name]
    for op, *args in edits:
        (delete if op == "del" else insert)(g, *args)
    assert violations(g) == bits
    with raks.Context(0) as ctx:
        with pytest.raises(raks.RaksError) as e:
            ctx.load_graph(g, alpha=0.5)
    assert e.value.code == -1
    assert int(re.search(r"bits (0x[0-9a-f]+)", str(e.value)).group(1), 16) == bits
