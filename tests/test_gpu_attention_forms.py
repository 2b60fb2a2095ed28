"""The forms of the bf16 attention kernel, each at sizes that choose it.

Small launches split a node's keys over the waves of a work-group; the unit
forms of 64, 128 and 256 queries take the rest, whole or with the last round's
units cut into key-range pieces.  Every case asserts the form that its plan
takes.  Plain inputs over overlapping windows; and, over windows of their own for
each node (whose pages a kernel then reads oldest chunk first), logits that rise
about 76 log2 units above the first key tile's maximum after the node's first
chunk: the waves then merge sums of very different scale, and the unit forms
pass their guard of 2^64 and redo the item exactly, which the test makes sure of
on the inputs.  Gates: the bf16 attention ones against the oracle, on sampled
rows.
"""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from oracle.attention import gather_context
from synth import TAG_V, normal
from synth.configs import Geometry

from gpu_cases import AttnCase, bf16_gates, sample_rows

pytestmark = pytest.mark.gpu


def _geo(heads, frames, gh, gw, W):
    return Geometry(heads=heads, head_dim=128, grid_h=gh, grid_w=gw, frames_per_chunk=frames, W=W)


WAVES = (32, 1, 1)
# name, geometry, nodes, form (queries per work-group, ring, pieces)
CASES = [
    ("waves-64x1344", _geo(2, 1, 8, 8, 20), 1, WAVES),      # 42 tiles over eight waves
    ("waves-page-ends", _geo(2, 1, 5, 8, 6), 3, WAVES),     # 40-token pages, 280 keys, a 24-key last tile
    ("waves-idle-wave", _geo(2, 1, 8, 9, 2), 1, WAVES),     # 216 keys: seven tiles, the last of 24 keys
    ("waves-ragged-q", _geo(3, 3, 8, 13, 3), 2, WAVES),     # 312 queries: a 24-query last work-group
    ("waves-128x512", _geo(12, 1, 8, 16, 3), 1, WAVES),
    ("unit-64", _geo(12, 1, 5, 8, 3), 32, (64, 4, 1)),
    ("unit-64-many", _geo(12, 1, 5, 8, 3), 64, (64, 3, 1)),
    ("unit-64-pieces", _geo(12, 1, 8, 8, 40), 3, (64, 4, 11)),
    ("unit-128", _geo(12, 1, 11, 24, 6), 3, (128, 2, 1)),   # nodes of 264 queries on 128-query units
    ("unit-128-pieces", _geo(2, 3, 8, 13, 6), 4, (128, 2, 7)),
    ("unit-256", _geo(7, 2, 20, 30, 3), 5, (256, 2, 1)),
    ("unit-256-pieces", _geo(3, 2, 20, 30, 1), 3, (256, 2, 5)),
]


def _redone(case, node, form, q_row=0, head=0):
    """Whether a unit form's item passes the guard: some key of it lies more than 64
    log2 units above the maximum of the item's first key tile."""
    tile, pieces = (32 if form[0] == 64 else 64), form[2]
    W = case.geo.W
    k, _ = gather_context([(case.pack[node][0] - r, 2) for r in range(W, -1, -1)], case.kv.__getitem__)
    s = k[:, head] @ case.q[node][q_row, head] * case.scale * np.log2(np.e)
    nt = -(-len(s) // tile)
    for p in range(pieces):
        part = s[p * nt // pieces * tile:(p + 1) * nt // pieces * tile]
        if part[tile:].size and part[tile:].max() - part[:tile].max() > 64:
            return True
    return False


@pytest.mark.parametrize("rising", [False, True], ids=["plain", "rising"])
@pytest.mark.parametrize("name,geo,nodes,form", CASES, ids=[c[0] for c in CASES])
def test_attention_forms(name, geo, nodes, form, rising):
    W = geo.W

    def key_fn(st, k):
        k = k.copy()
        k[:, :, 0] = 600.0 if st[0] % (W + 1) else 0.0
        return k

    def query_fn(st, q):
        q = q.copy()
        q[:, :, 0] = 1.0
        return q

    if rising:
        pack = [((W + 1) * i + W, 2) for i in range(nodes)]
        resident = [((W + 1) * i + r, 2) for i in range(nodes) for r in range(W)]
    else:
        pack = [(W + i, 2) for i in range(nodes)]
        resident = [(c, 2) for c in range(W)]
    case = AttnCase(geo, sc.SC_DTYPE_BF16, "same", pack, resident, seed=61,
                    key_fn=key_fn if rising else None, query_fn=query_fn if rising else None)
    assert sc.sc_attention_form(case.plan, case.cache) == form
    if rising and form != WAVES:
        assert all(_redone(case, i, form) for i in range(nodes))
    out = case.run()
    rows = sample_rows(geo.tokens_per_chunk, 24, seed=nodes)
    for i in range(0, nodes, 5 if nodes > 8 else 1):
        bf16_gates(out[i][rows], case.oracle(i, rows=rows), f"{name} node {pack[i]}")
    again = case.run()
    for i in range(nodes):
        assert np.array_equal(out[i], again[i])


@pytest.mark.parametrize("geo,nodes", [(_geo(2, 1, 5, 8, 6), 3), (_geo(2, 1, 8, 9, 4), 1), (_geo(2, 1, 8, 9, 6), 2)])
def test_waves_infinite_values(geo, nodes):
    """A channel of +inf in every value row stays +inf where a node's keys end
    inside the waves form's 32-key tile (280, 360 and 504 keys): the masked columns
    of that tile hold a real token's values at weight zero, and 0 x inf would be
    NaN.  The other channels stay right."""
    assert (geo.W + 1) * geo.tokens_per_chunk % 32 != 0

    def value_fn(st):
        v = normal((geo.tokens_per_chunk, geo.heads, geo.head_dim), (67, TAG_V) + tuple(st))
        v[:, :, 5] = np.inf
        return v

    pack = [(geo.W + i, 2) for i in range(nodes)]
    resident = [(c, 2) for c in range(geo.W)]
    case = AttnCase(geo, sc.SC_DTYPE_BF16, "same", pack, resident, seed=67, value_fn=value_fn)
    assert sc.sc_attention_form(case.plan, case.cache) == WAVES
    out = case.run()
    rest = np.arange(geo.head_dim) != 5
    for i in range(nodes):
        assert np.all(out[i][:, :, 5] == np.inf), i
        bf16_gates(out[i][:, :, rest], case.oracle(i)[:, :, rest], f"node {pack[i]}")
