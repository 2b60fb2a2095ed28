"""The fp32 attention at the sizes where its tiling can go wrong: pages of
half a key tile, pages ending inside one, fewer key tiles than waves, query
counts that are no multiple of a query tile, one and many nodes."""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from synth import normal
from synth.configs import Geometry

from gpu_cases import AttnCase, F32_MAX_ABS

pytestmark = pytest.mark.gpu

# Error model: u = 2^-24.  A logit of d products accumulated in any order is
# off by about sqrt(d) u times the products' scale (random signs), so by
# ~1e-6 at d = 128; the weights inherit it, the sum over keys averages it, and
# the output's own roundings are ~u.  Ten times that as a relative bound.
F32_REL = 1e-5


@pytest.mark.parametrize("heads,head_dim,grid,frames,window,kind,n", [
    (1, 64, (1, 8), 1, 0, "clean", 1),     # one half tile in all, 8 queries
    (3, 128, (1, 8), 3, 2, "same", 3),     # pages of half a tile
    (2, 64, (3, 8), 1, 2, "prog", 4),      # pages of one and a half tiles, 24 queries
    (2, 128, (8, 13), 3, 6, "prog", 5),    # 312 queries, 21 pages of 6.5 tiles
    (7, 128, (4, 4), 2, 5, "clean", 1),    # whole tiles, 12 of them over 8 waves
])
def test_f32_tiles(heads, head_dim, grid, frames, window, kind, n):
    dims = (44, 42, 42) if head_dim == 128 else (24, 20, 20)
    geo = Geometry(heads=heads, head_dim=head_dim, grid_h=grid[0], grid_w=grid[1], frames_per_chunk=frames,
                   K=4, W=window, rope_dims=dims)
    level = {"clean": lambda i: 4, "same": lambda i: 2, "prog": lambda i: i}[kind]
    pack = [(window + i, level(i)) for i in range(n)]
    resident = [(c, 2 if kind == "same" else 0) for c in range(window)]
    case = AttnCase(geo, sc.SC_DTYPE_F32, kind, pack, resident, seed=11)
    out = case.run()
    assert case.workspace_bytes == 0
    for i in range(n):
        want = case.oracle(i)
        assert np.abs(out[i] - want).max() <= F32_MAX_ABS, pack[i]
        assert np.linalg.norm(out[i] - want) <= F32_REL * np.linalg.norm(want), pack[i]


@pytest.mark.parametrize("head_dim,grid,frames", [(128, (8, 13), 3), (64, (1, 8), 1), (128, (5, 8), 2)])
def test_f32_infinite_values(head_dim, grid, frames):
    """A channel of +inf in every value row stays +inf where pages end inside a
    16-key tile: the masked half of that tile reads real tokens' values at
    weight zero, and 0 x inf would be NaN.  The other channels stay right."""
    geo = Geometry(heads=2, head_dim=head_dim, grid_h=grid[0], grid_w=grid[1], frames_per_chunk=frames, K=4, W=2,
                   rope_dims=(44, 42, 42) if head_dim == 128 else (24, 20, 20))
    assert geo.tokens_per_page % 16 == 8

    def value_fn(st):
        v = normal((geo.tokens_per_chunk, geo.heads, head_dim), (17, 3) + tuple(st))
        v[:, :, 5] = np.inf
        return v

    case = AttnCase(geo, sc.SC_DTYPE_F32, "same", [(2, 2), (3, 2)], [(0, 2), (1, 2)], seed=17, value_fn=value_fn)
    out = case.run()
    rest = np.arange(head_dim) != 5
    for i in range(2):
        assert np.all(out[i][:, :, 5] == np.inf), i
        want = case.oracle(i)[:, :, rest]
        assert np.abs(out[i][:, :, rest] - want).max() <= F32_MAX_ABS, i
