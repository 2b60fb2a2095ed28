"""K/V append over its element types, head dims and page sizes, rotated and not.

Pages of 8 tokens (one run), of 64 and 72 (a whole and a ragged block of 64)
and of three blocks; sources and pools that are only element-aligned.  Values
are moved, so bit-equal; keys take one rounding to the cache's type after the
rotation: 2^-8 of the largest (bf16: half a unit in the last place is 2^-9 of
the binade's top), 2^-21 (fp32: products and sums of values up to 2^3 rounded
thrice, and fp32 angles' cosines)."""
import numpy as np
import pytest

import paper_2609_22283_amd as sc
from oracle.rope import chunk_positions, rope
from synth import TAG_K, TAG_V, normal

from gpu_cases import to_device, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "shifted"])
@pytest.mark.parametrize("rotated", [False, True], ids=["raw", "rope"])
@pytest.mark.parametrize("gh,gw,frames", [(2, 4, 1), (8, 8, 2), (8, 9, 3), (9, 16, 1)])
@pytest.mark.parametrize("heads,hd", [(3, 128), (2, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_append(dtype, heads, hd, gh, gw, frames, rotated, shift):
    torch = torch_mod()
    code = sc.SC_DTYPE_BF16 if dtype == "bf16" else sc.SC_DTYPE_F32
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dims = (44, 42, 42) if hd == 128 else (24, 20, 20)
    tpp, n = gh * gw, gh * gw * frames
    args = (1, heads, hd, tpp, frames, 2 * frames, code)
    nbytes = sc.sc_cache_pool_bytes(*args)
    size = 2 if dtype == "bf16" else 4
    raw = torch.full((nbytes + 64,), 0xFF, dtype=torch.uint8, device="cuda")
    pool = raw[shift * size:shift * size + nbytes]
    cache = sc.sc_cache_create(pool, *args)
    table = torch.empty(sc.sc_rope_table_bytes(gh, gw, dims, 64), dtype=torch.uint8, device="cuda")
    rp = sc.sc_rope_table_build(table, gh, gw, dims, 64)
    for st in [(0, 0), (3, 1)]:
        src = []
        for tag in (TAG_K, TAG_V):
            t, vals = to_device(normal((n, heads, hd), (7, tag) + st), code)
            buf = torch.empty(t.numel() + 8, dtype=tdt, device="cuda")
            buf[shift:shift + t.numel()] = t.reshape(-1)
            src.append((buf[shift:shift + t.numel()], vals))
        (k, kv), (v, vv) = src
        cache.append(0, st, k, v, rope=rp if rotated else None)
        torch.cuda.synchronize()
        want = rope(kv, chunk_positions(st[0], frames, gh, gw), dims) if rotated else kv
        flat = torch.empty(nbytes // size, dtype=tdt, device="cuda")
        flat.view(torch.uint8).copy_(pool)
        pages = flat.view(2 * frames, 2, heads * tpp * hd).double().cpu().numpy()[cache.slots(st)]
        kg = pages[:, 0].reshape(frames, heads, tpp, hd).transpose(0, 2, 1, 3).reshape(n, heads, hd)
        vg = pages[:, 1].reshape(frames, heads, hd, tpp).transpose(0, 3, 1, 2).reshape(n, heads, hd)
        assert np.array_equal(vg, vv)
        if rotated:
            tol = (2.0 ** -8 if dtype == "bf16" else 2.0 ** -21) * np.abs(want).max()
            assert np.abs(kg - want).max() <= tol
        else:
            assert np.array_equal(kg, want)
    assert raw[shift * size + nbytes:].eq(0xFF).all() and raw[:shift * size].eq(0xFF).all()  # nothing outside the pool


@pytest.mark.parametrize("hd", [128, 64])
def test_append_rotation_bits(hd):
    """Rotated fp32 keys bit by bit: k0' = k0 c - [k1 s] and k1' = k0 s + [k1 c] with
    the bracketed product rounded to fp32 and the rest once (a fused multiply-add),
    so that cached keys stay the same from one build of the kernel to the next.
    In 64 bits that is a product and a sum of 24-bit values, rounded to fp32 at
    the end: the intermediate rounding at 53 bits changes the result only where
    it lands on a tie, about 2^-29 of the values."""
    torch = torch_mod()
    dims = (44, 42, 42) if hd == 128 else (24, 20, 20)
    heads, gh, gw, frames, chunk = 2, 5, 8, 2, 3
    tpp, n = gh * gw, gh * gw * frames
    args = (1, heads, hd, tpp, frames, frames, sc.SC_DTYPE_F32)
    pool = torch.full((sc.sc_cache_pool_bytes(*args),), 0xFF, dtype=torch.uint8, device="cuda")
    cache = sc.sc_cache_create(pool, *args)
    table = torch.empty(sc.sc_rope_table_bytes(gh, gw, dims, 64), dtype=torch.uint8, device="cuda")
    rp = sc.sc_rope_table_build(table, gh, gw, dims, 64)
    k, kv = to_device(normal((n, heads, hd), (7, TAG_K, 5)), sc.SC_DTYPE_F32)
    cache.append(0, (chunk, 0), k, k, rope=rp)
    torch.cuda.synchronize()
    cs = table.view(torch.float32).view(-1, 2).cpu().numpy()
    ends = np.cumsum([0, 64 * (dims[0] // 2), gh * (dims[1] // 2), gw * (dims[2] // 2)])
    axes = [cs[a:b].reshape(-1, d // 2, 2) for a, b, d in zip(ends, ends[1:], dims)]
    tok = np.arange(n)
    pos = [chunk * frames + tok // tpp, tok % tpp // gw, tok % gw]
    rot = np.concatenate([ax[p] for ax, p in zip(axes, pos)], 1)[:, None]  # [n, 1, hd / 2, 2]
    c, s = rot[..., 0], rot[..., 1]
    x0, x1 = kv[..., 0::2].astype(np.float32), kv[..., 1::2].astype(np.float32)
    r0 = x0.astype(np.float64) * c - (x1 * s).astype(np.float64)
    r1 = x0.astype(np.float64) * s + (x1 * c).astype(np.float64)
    want = np.stack([r0, r1], -1).reshape(n, heads, hd).astype(np.float32)
    got = pool.view(torch.float32).view(frames, 2, heads, tpp, hd)[:, 0].permute(0, 2, 1, 3).reshape(n, heads, hd)
    assert np.array_equal(got.cpu().numpy().view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("shift", [0, 2], ids=["aligned", "shifted"])
@pytest.mark.parametrize("k_norm", [False, True])
@pytest.mark.parametrize("heads,tpp,pages", [(2, 8, 1), (2, 72, 3), (12, 200, 1)])
def test_condition_pages(heads, tpp, pages, k_norm, shift):
    """A condition's K/V straight from the projections into its pages, in a pool
    that need not be 16-byte aligned: elementwise 2e-2 of max(1, |ref|) (two
    bf16 roundings of O(1) values)."""
    torch = torch_mod()
    D, L = heads * 128, tpp * pages
    args = (1, heads, 128, tpp, pages, 2 * pages, sc.SC_DTYPE_BF16)
    nbytes = sc.sc_cache_pool_bytes(*args)
    pool = torch.full((nbytes + 64,), 0xFF, dtype=torch.uint8, device="cuda")[shift:shift + nbytes]
    cache = sc.sc_cache_create(pool, *args)
    gen = torch.Generator(device="cuda").manual_seed(3)
    draw = lambda shape, s: (torch.randn(shape, generator=gen, device="cuda") * s).bfloat16()
    ctx, wk, wv = draw((L, D), 1.0), draw((D, D), D ** -0.5), draw((D, D), D ** -0.5)
    g = 1.0 + 0.3 * torch.randn(D, generator=gen, device="cuda") if k_norm else None
    nb = sc.sc_condition_workspace_bytes(cache)
    ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")
    for st in [(0, 0), (1, 0)]:
        sc.sc_condition_append(cache, 0, st, ctx, wk, wv, g, ws, nb)
    torch.cuda.synchronize()
    k, v = ctx.double() @ wk.double().T, ctx.double() @ wv.double().T
    if k_norm:
        k = k / (k.square().mean(-1, keepdim=True) + 1e-6).sqrt() * g.double()
    flat = torch.empty(nbytes // 2, dtype=torch.bfloat16, device="cuda")
    flat.view(torch.uint8).copy_(pool)
    for st in [(0, 0), (1, 0)]:
        got = flat.view(2 * pages, 2, -1).double()[torch.tensor(cache.slots(st), device="cuda")]
        kg = got[:, 0].view(pages, heads, tpp, 128).permute(0, 2, 1, 3).reshape(L, D)
        vg = got[:, 1].view(pages, heads, 128, tpp).permute(0, 3, 1, 2).reshape(L, D)
        for a, ref in ((kg, k), (vg, v)):
            assert ((a - ref).abs() / ref.abs().clamp(min=1.0)).max().item() <= 2e-2
