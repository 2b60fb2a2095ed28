"""The forms of the bf16 attention kernel, each at sizes that choose it.

Small launches split a node's keys over the waves of a work-group; the unit
forms of 64, 128 and 256 queries take the rest.  Plain inputs, and logits that
rise far above the first key tile's maximum (about 76 log2 units from the third
chunk on: the waves then merge sums of very different scale, and the unit forms
redo their items exactly).  Gates: the bf16 attention ones against the oracle,
on sampled rows.
"""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from synth import TAG_V, normal
from synth.configs import Geometry

from gpu_cases import AttnCase, bf16_gates, sample_rows

pytestmark = pytest.mark.gpu


def _geo(heads, frames, gh, gw, W):
    return Geometry(heads=heads, head_dim=128, grid_h=gh, grid_w=gw, frames_per_chunk=frames, W=W)


# name, geometry, nodes
CASES = [
    ("waves-64x1344", _geo(2, 1, 8, 8, 20), 1),       # 42 tiles over eight waves
    ("waves-page-ends", _geo(2, 1, 5, 8, 6), 3),      # 40-token pages, 280 keys, a 24-key last tile
    ("waves-one-tile", _geo(1, 1, 4, 8, 0), 1),       # 32 keys: seven waves without a tile
    ("waves-ragged-q", _geo(3, 3, 8, 13, 3), 2),      # 312 queries: a 24-query last work-group
    ("waves-128x512", _geo(12, 1, 8, 16, 3), 1),
    ("unit-64", _geo(12, 1, 5, 8, 3), 32),
    ("unit-128", _geo(12, 1, 11, 24, 6), 3),          # nodes of 264 queries on 128-query units
    ("unit-256", _geo(7, 2, 20, 30, 3), 5),
]


@pytest.mark.parametrize("rising", [False, True], ids=["plain", "rising"])
@pytest.mark.parametrize("name,geo,nodes", CASES, ids=[c[0] for c in CASES])
def test_attention_forms(name, geo, nodes, rising):
    def key_fn(st, k):
        k = k.copy()
        k[:, :, 0] = 600.0 if st[0] >= 2 else 0.0
        return k

    def query_fn(st, q):
        q = q.copy()
        q[:, :, 0] = 1.0
        return q

    pack = [(geo.W + i, 2) for i in range(nodes)]
    resident = [(c, 2) for c in range(geo.W)]
    case = AttnCase(geo, sc.SC_DTYPE_BF16, "same", pack, resident, seed=61,
                    key_fn=key_fn if rising else None, query_fn=query_fn if rising else None)
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
    out = case.run()
    rest = np.arange(geo.head_dim) != 5
    for i in range(nodes):
        assert np.all(out[i][:, :, 5] == np.inf), i
        bf16_gates(out[i][:, :, rest], case.oracle(i)[:, :, rest], f"node {pack[i]}")
