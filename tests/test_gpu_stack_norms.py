"""A stack's folded RMSNorms: layer by layer against the single block.

Inside sc_stack_forward a layer without modulation takes its first RMSNorm from
the sums of squares that the layer before stored with its rows; a block called by
itself takes it from a pass over the rows.  Both are the same factor up to the
order of an fp32 sum, so the two results differ only where that moves a bf16
rounding.  Rows of very different size (2^-3 .. 2^3) make a factor of another row
or of another layer's rows show.

Gate.  Either result is within a few roundings of 2^-9 of the exact one per layer
(0.0026 - 0.0034 in the 2-norm, measured for one block), so two of them are
within 2 * 0.0034 per layer of each other; a wrong factor moves whole rows by at
least a factor of two.  A layer with a cross-attention carries one more branch of
the same kind: twice the distance.
"""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from synth import (TAG_CTX, TAG_W_CK, TAG_W_CO, TAG_W_CQ, TAG_W_CV, TAG_W_DOWN, TAG_W_O, TAG_W_QKV, TAG_W_UP, TAG_X,
                   normal, normal_parallel)

from gpu_cases import to_device, torch_mod

pytestmark = pytest.mark.gpu
DIMS = (44, 42, 42)

# heads (256, 1536 and 2304 features: 1, 6 and 9 runs of partials per row), nodes, grid, modulated layers,
# layers with a cross-attention
CASES = [
    (2, 1, 8, 9, (), ()), (2, 3, 8, 13, (1,), ()), (12, 1, 8, 8, (), ()), (12, 3, 8, 9, (0,), ()),
    (18, 2, 8, 9, (), ()), (18, 1, 8, 11, (2,), ()), (2, 2, 30, 52, (), ()),
    (12, 1, 4, 8, (), ()), (18, 1, 8, 8, (), ()),
    (2, 2, 8, 13, (), (0, 1, 2)), (2, 2, 8, 13, (1,), (0, 1)), (12, 1, 4, 8, (), (0, 1, 2)),
]
# (heads, tokens) at which QKV's contraction is split: the reduce kernel makes the factors from the sums
SPLIT_QKV = {(12, 32), (18, 64)}


@pytest.mark.parametrize("qk", [False, True], ids=["plain", "qk"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_stack_against_single_blocks(case, qk):
    torch = torch_mod()
    heads, n_nodes, gh, gw, modulated, crossed = case
    D, mlp, tpp, layers = heads * 128, 512, gh * gw, 3
    T, nodes = n_nodes * tpp, [(i, i) for i in range(n_nodes)]
    assert (sc.sc_gemm_form("gemm_qkv", 3 * D, T, D)[3] > 1) == ((heads, T) in SPLIT_QKV)
    gen = lambda shape, tag, s: to_device(normal_parallel(shape, (93, tag), s), sc.SC_DTYPE_BF16)[0]
    stack = []
    for l in range(layers):
        mod = None
        if l in modulated:
            m = normal((5, 6, D), (93, 30 + l), 0.2).astype(np.float32)
            m[:, 2] += 1.0
            m[:, 5] += 1.0
            mod = torch.from_numpy(m).cuda()
        g = torch.from_numpy((1.0 + 0.3 * normal((2, D), (93, 40 + l))).astype(np.float32)).cuda() if qk else None
        stack.append(sc.BlockWeights(
            D, heads, 128, mlp, gen((3 * D, D), TAG_W_QKV + 100 * l, 0.02), gen((D, D), TAG_W_O + 100 * l, 0.02),
            gen((mlp, D), TAG_W_UP + 100 * l, 0.02), gen((D, mlp), TAG_W_DOWN + 100 * l, 0.02), mod=mod, qk_norm=g))
    if crossed:
        L, f32 = 72, lambda shape, tag: torch.from_numpy((1.0 + 0.3 * normal(shape, (93, tag))).astype(np.float32)).cuda()
        args = (layers, heads, 128, L, 1, 1, sc.SC_DTYPE_BF16)
        cond_pool = torch.zeros(sc.sc_cache_pool_bytes(*args), dtype=torch.uint8, device="cuda")
        cond = sc.sc_cache_create(cond_pool, *args)
        nb = sc.sc_condition_workspace_bytes(cond)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        mats = {l: [gen((D, D), tag + 100 * l, D ** -0.5) for tag in (TAG_W_CK, TAG_W_CV, TAG_W_CQ, TAG_W_CO)]
                for l in crossed}
        for l in crossed:
            sc.sc_condition_append(cond, l, (0, 0), gen((L, D), TAG_CTX, 1.0), mats[l][0], mats[l][1],
                                   f32((D,), 50 + l), ws, nb)
        plan_c = sc.sc_plan_condition(cond, [(0, 0)] * n_nodes, tpp)
        for l in crossed:
            stack[l] = stack[l].with_cross(sc.CrossAttn(mats[l][2], mats[l][3], cond, plan_c,
                                                        q_norm=f32((D,), 60 + l) if l else None))
    x = gen((T, D), TAG_X, 1.0)
    x *= 2.0 ** (torch.arange(T, device="cuda") % 7 - 3)[:, None].to(x.dtype)
    table = torch.empty(sc.sc_rope_table_bytes(gh, gw, DIMS, 64), dtype=torch.uint8, device="cuda")
    rp = sc.sc_rope_table_build(table, gh, gw, DIMS, 64)
    nb = sc.sc_block_workspace_bytes(stack[0], T)

    def run(together):
        args = (layers, heads, 128, tpp, 1, n_nodes, sc.SC_DTYPE_BF16)
        pool = torch.full((sc.sc_cache_pool_bytes(*args),), 0xFF, dtype=torch.uint8, device="cuda")
        cache = sc.sc_cache_create(pool, *args)
        plan = sc.sc_plan_build(sc.sc_selection_build("prog", 4, 0, nodes), cache)
        ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")
        y = x.clone()
        if together:
            sc.sc_stack_forward(stack, cache, plan, y, rp, ws, nb)
        else:
            for l, w in enumerate(stack):
                sc.sc_block_forward(w, cache, l, plan, y, rp, ws, nb)
        torch.cuda.synchronize()
        return y.double(), pool.view(torch.bfloat16).view(layers, -1).double()

    (y, kv), (y1, kv1) = run(True), run(False)
    per_layer = 2 * 0.0034 * (2 if crossed else 1)
    for a, b, n in [(y, y1, layers)] + [(kv[l], kv1[l], l + 1) for l in range(layers)]:
        assert torch.isfinite(a).all()
        assert ((a - b).norm() / b.norm()).item() <= per_layer * n
    rows = (y - y1).norm(dim=1) / y1.norm(dim=1)
    assert rows.max().item() <= 4 * per_layer * layers
