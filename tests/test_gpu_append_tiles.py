"""The prefill append at shapes that take each tile of its GEMM, with ragged token counts and a column count that is no
multiple of the tile's width, every appended row against a float64 product on the same inputs.  Bound: 2e-2, max-abs-rel."""
import pytest
import torch

import paper_2503_01586_amd as ekv
from gpu_util import DEV, TOL, gpu_append

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r,d_c,T", [
    (2048, 8, 1408, 8100),      # 256 x 256, four waves; 1920 columns: the last block overlaps the one before
    (2048, 8, 1536, 8192),      # ... whole blocks
    (1024, 8, 1408, 8100),      # 256 x 256, eight waves
    (1024, 8, 1536, 4000),      # 256 x 128
    (1024, 8, 1536, 2000),      # 128 x 128, two contraction groups
    (1024, 4, 768, 130),        # 64 x 128
    (32, 8, 1536, 8100),        # one stage of contraction rows
    (160, 8, 1408, 8100),       # as many stages as the ring holds
    (1000, 8, 1536, 300),       # rows that are no whole stages: the register-staged kernel
])
def test_append_tiles(d, r, d_c, T):
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
