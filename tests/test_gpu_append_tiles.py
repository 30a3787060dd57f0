"""The prefill append and the rebuild of keys and values at shapes that take each tile of their GEMM, with ragged token
counts, a column count that is no multiple of the tile's width, and contractions shorter than, equal to and longer than
the tile's ring of stages (32 rows each), every row against a float64 product on the same inputs.
Bound: 2e-2, max-abs-rel."""
import pytest
import torch

import paper_2503_01586_amd as ekv
from gpu_util import DEV, TOL, gpu_append

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r,d_c,T,tile", [
    (2048, 8, 1408, 8100, ekv.TILE_256_256_WIDE),    # 1920 columns: the last block overlaps the one before
    (2048, 8, 1536, 8192, ekv.TILE_256_256_WIDE),    # ... whole blocks
    (1024, 8, 1408, 8100, ekv.TILE_256_256),
    (1024, 8, 1536, 4000, ekv.TILE_128_128_PAIRS),
    (1024, 8, 1536, 2000, ekv.TILE_128_128),
    (1024, 4, 768, 130, ekv.TILE_64_128),
    (32, 8, 1536, 8100, ekv.TILE_128_128_PAIRS),     # one stage of contraction rows
    (160, 8, 1408, 8100, ekv.TILE_128_128_PAIRS),    # one more than the ring holds
    (1000, 8, 1536, 300, ekv.TILE_STAGED_64_128),    # rows that are no whole stages
    (40, 8, 7680, 4000, ekv.TILE_STAGED_256_128),
])
def test_append_tiles(d, r, d_c, T, tile):
    n_h, d_h = 32, 128
    g = torch.Generator(device=DEV)
    g.manual_seed(d + T)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device=DEV) * std).bfloat16()
    x, W_ke, W_d = normal(T, d), normal(d, n_h, 2 * r, std=d ** -0.5), normal(d, d_c, std=d ** -0.5)
    idx = torch.stack([torch.randperm(d_h // 2, generator=g, device=DEV)[:r] for _ in range(n_h)]).int()
    pos = torch.randint(0, 30000, (T,), generator=g, device=DEV, dtype=torch.int32)
    slot = torch.randperm(T + 7, generator=g, device=DEV)[:T]
    slot[T // 3] = -1                                        # skipped
    dims = ekv.make_dims(d, n_h, d_h, r, d_c, "bf16")
    assert ekv.elitekv_append_gemm_tile(dims, T) == tile
    ke = torch.full((T + 7, n_h, 2 * r), 7.0, dtype=torch.bfloat16, device=DEV)
    c = torch.full((T + 7, d_c), 7.0, dtype=torch.bfloat16, device=DEV)
    gpu_append(dims, x, pos, slot, W_ke, W_d, idx, T + 7, ke, c)
    keep = slot >= 0
    ref_c = x.double() @ W_d.double()
    y = (x.double() @ W_ke.double().reshape(d, -1)).reshape(T, n_h, r, 2)
    a = pos.double()[:, None, None] * (10000.0 ** (-2.0 * idx.double() / d_h))[None]
    ref_ke = torch.stack((y[..., 0] * a.cos() - y[..., 1] * a.sin(), y[..., 0] * a.sin() + y[..., 1] * a.cos()), dim=3)
    for got, ref in ((c[slot[keep]], ref_c[keep]), (ke[slot[keep]], ref_ke.reshape(T, n_h, 2 * r)[keep])):
        assert float((got.double() - ref).abs().max() / ref.abs().max()) <= TOL["bf16"]
    untouched = torch.ones(T + 7, dtype=torch.bool, device=DEV)
    untouched[slot[keep]] = False
    assert bool((c[untouched] == 7.0).all()) and bool((ke[untouched] == 7.0).all())


@pytest.mark.parametrize("d_ck,d_cv,S,tile", [
    # separated latents: the tile is chosen by the longer contraction, the other one is short; 3840 columns
    (32, 3072, 3000, ekv.TILE_256_256_WIDE),         # one stage; the ring holds five
    (96, 3072, 3000, ekv.TILE_256_256_WIDE),
    (160, 3072, 4000, ekv.TILE_256_256_WIDE),
    (192, 3072, 4000, ekv.TILE_256_256_WIDE),
    (3072, 128, 3001, ekv.TILE_256_256_WIDE),        # the values' columns have the short one
    (32, 1024, 3000, ekv.TILE_256_256),              # one stage; the ring holds four
    (96, 1024, 3000, ekv.TILE_256_256),
    (128, 1024, 4000, ekv.TILE_256_256),
    (1024, 160, 4000, ekv.TILE_256_256),
    (96, 1024, 1501, ekv.TILE_128_128_PAIRS),        # four
    (1024, 192, 1501, ekv.TILE_128_128_PAIRS),
    (64, 1024, 1000, ekv.TILE_128_128),              # the rings of the other tiles hold six
    (1024, 224, 1000, ekv.TILE_128_128),
    (96, 1024, 201, ekv.TILE_64_128),
    (32, 512, 200, ekv.TILE_64_128),
])
def test_rebuild_tiles(d_ck, d_cv, S, tile):
    """The rebuilt rows, which the call leaves in its workspace: [keys without their elite dims | values] of every head."""
    n_h, d_h, r, T = 16, 128, 8, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(d_ck + S)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device=DEV) * std).bfloat16()
    dims = ekv.make_dims(64, n_h, d_h, r, d_ck + d_cv, "bf16")
    assert ekv.elitekv_prefill_gemm_tile(dims, T, S, d_ck) == tile
    W_uk, W_uv = normal(d_ck, n_h, d_h - 2 * r, std=d_ck ** -0.5), normal(d_cv, n_h, d_h, std=d_cv ** -0.5)
    q, ke, c = normal(1, T, n_h, d_h), normal(S, n_h, 2 * r), normal(S, d_ck + d_cv)
    idx = torch.stack([torch.randperm(d_h // 2, generator=g, device=DEV)[:r] for _ in range(n_h)]).int()
    pos = torch.arange(S - T, S, device=DEV, dtype=torch.int32)
    out = torch.full_like(q, float("nan"))
    ws = torch.full((ekv.elitekv_slrd_prefill_attn_workspace_bytes(dims, d_ck, 1, T, S),), 0xFF, dtype=torch.uint8, device=DEV)
    ekv.elitekv_slrd_prefill_attn(dims, d_ck, q, pos.reshape(1, T), (pos + 1).reshape(1, T), S, S, W_uk, W_uv, idx, ke, c, out, ws)
    torch.cuda.synchronize()
    n_k = n_h * (d_h - 2 * r)
    kv = ws.view(torch.bfloat16)[:S * (n_k + n_h * d_h)].reshape(S, -1).double()
    keys = c[:, :d_ck].double() @ W_uk.double().reshape(d_ck, -1)
    values = c[:, d_ck:].double() @ W_uv.double().reshape(d_cv, -1)
    for got, ref in ((kv[:, :n_k], keys), (kv[:, n_k:], values)):
        assert float((got - ref).abs().max() / ref.abs().max()) <= TOL["bf16"]
    assert bool(torch.isfinite(out).all())
