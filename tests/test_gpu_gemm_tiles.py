"""The block's GEMMs over the sizes where their tile shape changes.

launch_gemm picks one of eight tile shapes and a split of the contraction by
size; the packs below (window 0: every node attends to itself) make the four
projections take each of them, which every case asserts, with token counts that end inside a tile and
inside a 16-token block, and contractions whose parts differ by a stage.  The
expected block is plain torch in 64 bits on the same bf16 inputs.

Gates.  The residual stream is rounded to bf16 twice, as x' = x + a and as
the output y, each moving a value by at most 2^-8 of it.  The MLP branch (rms
about 1, times a gate of up to 1.8 where modulated) carries the roundings of
x', of its normalised input (1536 terms each) and of the GELU output (8960
terms), independent errors of at most 2^-8 / sqrt(12) of a term in the rms:
six standard deviations of the three together are 6 sqrt(3) 2^-8 / sqrt(12)
1.8 = 0.021.  So |d| <= 2^-8 (|x'| + |y|) + 2.1e-2 per element, and the block
gate 4e-3 max(1, mean |ref|) in the mean, which is the sharper of the two: a
tile or a part of a contraction that goes wrong moves whole rows.  The K/V
pages carry up to two roundings of O(1) values: 2e-2 of max(1, |ref|) per
element.
"""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from oracle.rope import chunk_positions, rope
from synth import TAG_GAIN, TAG_W_DOWN, TAG_W_O, TAG_W_QKV, TAG_W_UP, TAG_X, normal, normal_parallel

from gpu_cases import to_device, torch_mod

pytestmark = pytest.mark.gpu
DIMS, EPS = (44, 42, 42), 1e-6

# (tile features, tile tokens, ring)
T64, T128X64, T128, T128D = (64, 64, 5), (128, 64, 3), (128, 128, 2), (128, 128, 4)
T256X128, T192, T224, T256 = (256, 128, 3), (256, 192, 2), (256, 224, 2), (256, 256, 2)
# heads, mlp, nodes, frames, grid_h, grid_w: the tile and parts of QKV, out, up, down
SIZES = {
    (12, 8960, 1, 1, 4, 8): [(T128X64, 6), (T64, 8), (T64, 1), (T64, 10)],             # 32 tokens
    (12, 8960, 1, 1, 8, 9): [(T64, 1), (T64, 1), (T128X64, 1), (T128X64, 10)],         # 72
    (12, 8960, 2, 1, 8, 13): [(T128X64, 1), (T64, 1), (T128D, 1), (T128D, 10)],        # 208
    (12, 8960, 1, 2, 11, 24): [(T128D, 1), (T64, 1), (T256X128, 1), (T128D, 4)],       # 528
    (12, 8960, 1, 1, 25, 40): [(T128, 1), (T128X64, 1), (T192, 1), (T256X128, 5)],     # 1000
    (12, 8960, 1, 3, 25, 40): [(T224, 1), (T256X128, 1), (T224, 1), (T224, 3)],        # 3000
    (12, 8960, 4, 3, 29, 40): [(T128, 1), (T192, 1), (T256, 1), (T192, 1)],            # 13920
    (6, 3072, 1, 1, 8, 17): [(T128X64, 1), (T64, 1), (T64, 1), (T64, 7)],              # 136
}


def _rms(x):
    return x / (x.square().mean(-1, keepdim=True) + EPS).sqrt()


@pytest.mark.parametrize("full", [False, True], ids=["plain", "mod-qk"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "-".join(map(str, s)))
def test_block_over_gemm_tiles(size, full):
    torch = torch_mod()
    heads, mlp, n_nodes, frames, gh, gw = size
    hd, tpp, n = 128, gh * gw, frames * gh * gw
    D, T = heads * 128, n_nodes * frames * gh * gw
    for (tile, parts), (kind, f, k) in zip(SIZES[size], [("gemm_qkv", 3 * D, D), ("gemm_out", D, D),
                                                         ("gemm_up", mlp, D), ("gemm_down", D, mlp)]):
        assert sc.sc_gemm_form(kind, f, T, k) == tile + (parts,)
    nodes = [(i, i) for i in range(n_nodes)]
    gen = lambda shape, tag, s: to_device(normal_parallel(shape, (91, tag), s), sc.SC_DTYPE_BF16)[0]
    w = {"w_qkv": gen((3 * D, D), TAG_W_QKV, 0.02), "w_o": gen((D, D), TAG_W_O, 0.02),
         "w_up": gen((mlp, D), TAG_W_UP, 0.02), "w_down": gen((D, mlp), TAG_W_DOWN, 0.02)}
    x = gen((T, D), TAG_X, 1.0)
    mod = qk = None
    if full:
        m = normal((5, 6, D), (91, 30), 0.2).astype(np.float32)
        m[:, 2] += 1.0
        m[:, 5] += 1.0
        mod = torch.from_numpy(m).cuda()
        qk = torch.from_numpy((1.0 + 0.3 * normal((2, D), (91, TAG_GAIN))).astype(np.float32)).cuda()
    args = (1, heads, hd, tpp, frames, n_nodes * frames, sc.SC_DTYPE_BF16)
    pool = torch.full((sc.sc_cache_pool_bytes(*args),), 0xFF, dtype=torch.uint8, device="cuda")
    cache = sc.sc_cache_create(pool, *args)
    table = torch.empty(sc.sc_rope_table_bytes(gh, gw, DIMS, 64), dtype=torch.uint8, device="cuda")
    rp = sc.sc_rope_table_build(table, gh, gw, DIMS, 64)
    weights = sc.BlockWeights(D, heads, hd, mlp, w["w_qkv"], w["w_o"], w["w_up"], w["w_down"], mod=mod, qk_norm=qk)
    plan = sc.sc_plan_build(sc.sc_selection_build("prog", 4, 0, nodes), cache)
    nb = sc.sc_block_workspace_bytes(weights, T)
    ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")
    y = x.clone()
    sc.sc_block_forward(weights, cache, 0, plan, y, rp, ws, nb)
    torch.cuda.synchronize()

    w = {k: v.double() for k, v in w.items()}
    pages = pool.view(torch.bfloat16).view(n_nodes * frames, 2, heads * tpp * hd).double()
    for i, (c, j) in enumerate(nodes):
        xi = x[i * n:(i + 1) * n].double()
        lev = mod[j].double() if full else None
        norm = lambda v, k: _rms(v) * (1 + lev[3 * k + 1]) + lev[3 * k] if full else _rms(v)
        q, k, v = (norm(xi, 0) @ w["w_qkv"].T).split(D, 1)
        if full:
            q, k = _rms(q) * qk[0].double(), _rms(k) * qk[1].double()
        pos = chunk_positions(c, frames, gh, gw)
        q, k = (torch.from_numpy(rope(a.view(n, heads, hd).cpu().numpy(), pos, DIMS)).cuda() for a in (q, k))
        v = v.view(n, heads, hd)
        got = pages[torch.tensor(cache.slots((c, j)), device="cuda")]
        kp = got[:, 0].view(frames, heads, tpp, hd).permute(0, 2, 1, 3).reshape(n, heads, hd)
        vp = got[:, 1].view(frames, heads, hd, tpp).permute(0, 3, 1, 2).reshape(n, heads, hd)
        for name, a, ref in (("k", kp, k), ("v", vp, v)):
            bad = (a - ref).abs() / ref.abs().clamp(min=1.0)
            assert bad.max().item() <= 2e-2, (name, i, bad.max().item())
        o = torch.stack([torch.softmax(q[:, h] @ k[:, h].T * hd ** -0.5, -1) @ v[:, h] for h in range(heads)], 1)
        a = o.reshape(n, D) @ w["w_o"].T
        xi = xi + (lev[2] * a if full else a)
        f = torch.nn.functional.gelu(norm(xi, 1) @ w["w_up"].T, approximate="tanh") @ w["w_down"].T
        ref = xi + (lev[5] * f if full else f)
        err = (y[i * n:(i + 1) * n].double() - ref).abs()
        over = (err - (xi.abs() + ref.abs()) * 2.0 ** -8).max().item()
        assert over <= 2.1e-2, (i, over)
        assert err.mean().item() <= 4e-3 * max(1.0, ref.abs().mean().item())
