"""GPU parity of the matrix-core front launch, query preparation and batched merge where they begin and where a block of
theirs is not full: from two sequences on, and latent widths that are odd multiples of 64 columns on either side of a
separated latent.  Shapes outside those kernels (a hidden width that is no multiple of eight) keep the vector-unit ones.
Against the float64 oracle, through the C ABI; bound max-abs-rel <= 2e-2 (bf16)."""
import numpy as np
import pytest
import torch

import elitekv_synth as synth
import paper_2503_01586_amd as ekv
from oracle import elitekv_oracle as orc

from gpu_util import DEV, TOL, dev, dims_of, gpu_append, gpu_decode, host64, i32, i64
from test_gpu_parity import _draw, shape
from test_gpu_slrd import _draw as _draw_slrd, gpu_slrd_decode, shape as slrd_shape

pytestmark = pytest.mark.gpu

# (d_model, heads, head_dim, r, d_ck, d_cv)
SEPARATED = [(136, 8, 64, 4, 192, 192), (256, 32, 128, 8, 320, 320), (192, 40, 128, 4, 448, 448), (512, 32, 128, 8, 576, 960)]


def _slrd_planes(sh, rng, B, stride):
    ke, c = synth.draw_cache_planes(rng, B * stride, sh["n_heads"], sh["r"], sh["d_c"])
    return dev(ke, "bf16"), dev(c, "bf16")


def _latents(c, B, sh):
    c = c.reshape(B, -1, sh["d_c"])
    return c[..., :sh["d_ck"]], c[..., sh["d_ck"]:]


@pytest.mark.parametrize("B", [2, 3, 7, 9, 33])
@pytest.mark.parametrize("dims6", SEPARATED, ids=lambda t: "%d+%d" % t[4:])
def test_separated_step(dims6, B):
    sh = slrd_shape(*dims6, "bf16")
    seqs = [1 + (37 * i + 15) % 83 for i in range(B)]
    stride, n_h, d_h, d_ck = max(seqs) + 2, sh["n_heads"], sh["head_dim"], sh["d_ck"]
    rng, idx, W_ke, A_k, A_v, B_k, B_v, x, q = _draw_slrd(sh, B, B, 40 + B)
    dims = dims_of(sh)
    ke, c = _slrd_planes(sh, rng, B, stride)
    pos = np.array(seqs) - 1
    slot = np.arange(B) * stride + pos
    xd, qd, Wked, Akd, Avd, Bkd, Bvd = (dev(a, "bf16") for a in (x, q, W_ke, A_k, A_v, B_k, B_v))
    out = torch.full((B, n_h, d_h), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ekv.elitekv_slrd_decode_step_workspace_bytes(dims, d_ck, B, max(seqs)),), 0xFF, dtype=torch.uint8, device=DEV)
    ekv.elitekv_slrd_decode_step(dims, d_ck, xd, qd, i32(pos), i64(slot), i32(seqs), max(seqs), stride, Wked, Akd, Avd, Bkd, Bvd,
                                 i32(idx), ke, c, out, ws)
    torch.cuda.synchronize()
    ke_ref, ck_ref, cv_ref = orc.slrd_append(host64(xd), pos, host64(Wked), host64(Akd), host64(Avd), idx, d_h, sh["rope_base"])
    c_ref = np.concatenate([ck_ref, cv_ref], axis=1)
    ke_g, c_g = host64(ke).reshape(B * stride, n_h, -1), host64(c)
    assert orc.max_abs_rel(c_g[slot], c_ref) <= TOL["bf16"]
    assert orc.max_abs_rel(ke_g[slot], ke_ref) <= TOL["bf16"]
    ref = orc.slrd_decode_attn(host64(qd), pos, ke_g.reshape(B, stride, n_h, -1), *_latents(c_g, B, sh), seqs, host64(Bkd),
                               host64(Bvd), idx, d_h, sh["rope_base"])
    assert orc.max_abs_rel(host64(out), ref) <= TOL["bf16"]


@pytest.mark.parametrize("n_splits", [1, 5])
@pytest.mark.parametrize("dims6", SEPARATED, ids=lambda t: "%d+%d" % t[4:])
def test_separated_decode(dims6, n_splits):
    sh = slrd_shape(*dims6, "bf16")
    seqs = [70, 0, 33]                                     # with a sequence that attends to nothing
    B, stride, d_ck = len(seqs), 72, sh["d_ck"]
    rng, idx, _, _, _, B_k, B_v, _, q = _draw_slrd(sh, 1, B, 60)
    dims = dims_of(sh)
    ke, c = _slrd_planes(sh, rng, B, stride)
    qd, Bkd, Bvd = (dev(a, "bf16") for a in (q, B_k, B_v))
    pos = np.maximum(np.array(seqs) - 1, 0)
    out = gpu_slrd_decode(dims, d_ck, qd, i32(pos), i32(seqs), max(seqs), stride, Bkd, Bvd, i32(idx), ke, c, n_splits)
    ref = orc.slrd_decode_attn(host64(qd), pos, host64(ke).reshape(B, stride, sh["n_heads"], -1), *_latents(host64(c), B, sh),
                               seqs, host64(Bkd), host64(Bvd), idx, sh["head_dim"], sh["rope_base"])
    assert orc.max_abs_rel(host64(out), ref) <= TOL["bf16"]
    assert torch.count_nonzero(out[1]) == 0


@pytest.mark.parametrize("B, n_h", [(1, 32), (3, 32), (7, 32), (8, 32), (8, 40)])     # eight: every sequence on one XCD
def test_hidden_width_outside_the_matrix_core_front(B, n_h):
    sh = shape(1004, n_h, 128, 8, 512, "bf16")             # rows of x are not 16-byte aligned
    seqs = [5 + 13 * i for i in range(B)]
    stride, d_h = max(seqs) + 1, 128
    rng, idx, W_ke, W_dkv, W_uk, W_uv, x, q = _draw(sh, B, B, 80 + B)
    dims = dims_of(sh)
    ke64, c64 = synth.draw_cache_planes(rng, B * stride, n_h, 8, 512)
    ke, c = dev(ke64, "bf16"), dev(c64, "bf16")
    pos = np.array(seqs) - 1
    slot = np.arange(B) * stride + pos
    xd, qd, Wked, Wdkvd, Wukd, Wuvd = (dev(a, "bf16") for a in (x, q, W_ke, W_dkv, W_uk, W_uv))
    out = torch.full((B, n_h, d_h), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ekv.elitekv_decode_step_workspace_bytes(dims, B, max(seqs)),), 0xFF, dtype=torch.uint8, device=DEV)
    ekv.elitekv_decode_step(dims, xd, qd, i32(pos), i64(slot), i32(seqs), max(seqs), stride, Wked, Wdkvd, Wukd, Wuvd, i32(idx), ke,
                            c, out, ws)
    torch.cuda.synchronize()
    ke_ref, c_ref = orc.append(host64(xd), pos, host64(Wked), host64(Wdkvd), idx, d_h, sh["rope_base"])
    ke_g, c_g = host64(ke).reshape(B * stride, n_h, -1), host64(c)
    assert orc.max_abs_rel(c_g[slot], c_ref) <= TOL["bf16"]
    assert orc.max_abs_rel(ke_g[slot], ke_ref) <= TOL["bf16"]
    ref = orc.decode_attn(host64(qd), pos, ke_g.reshape(B, stride, n_h, -1), c_g.reshape(B, stride, -1), seqs, host64(Wukd),
                          host64(Wuvd), idx, d_h, sh["rope_base"])
    assert orc.max_abs_rel(host64(out), ref) <= TOL["bf16"]


@pytest.mark.parametrize("T", [1, 2, 3, 7, 8])
@pytest.mark.parametrize("d_model", [64, 136, 4096])       # less than a stage of the contraction, a ragged one, whole ones
def test_append_of_few_tokens(d_model, T):
    sh = shape(d_model, 32, 128, 8, 1536, "bf16")
    rng, idx, W_ke, W_dkv, _, _, x, _ = _draw(sh, T, 1, 100 + T)
    dims = dims_of(sh)
    pos = np.array([3 * t + 11 for t in range(T)])
    slot = np.array([T - 1 - t for t in range(T)])
    xd, Wked, Wdkvd = (dev(a, "bf16") for a in (x, W_ke, W_dkv))
    ke, c = gpu_append(dims, xd, i32(pos), i64(slot), Wked, Wdkvd, i32(idx), T)
    ke_ref, c_ref = orc.append(host64(xd), pos, host64(Wked), host64(Wdkvd), idx, 128, sh["rope_base"])
    assert orc.max_abs_rel(host64(c)[slot], c_ref) <= TOL["bf16"]
    assert orc.max_abs_rel(host64(ke).reshape(T, 32, -1)[slot], ke_ref) <= TOL["bf16"]


# every chunk width of the one-row merge, the batched merge for a single row (a width of neither), more splits than one pass
# of either takes, and row tiles cut down to the weights the LDS holds
@pytest.mark.parametrize("B, n_splits", [(1, 1), (1, 300), (1, 1024), (9, 1024)])
@pytest.mark.parametrize("n_h, d_ck, d_c", [(32, 0, 128), (32, 0, 768), (32, 0, 1024), (32, 0, 1536), (40, 0, 1920), (32, 320, 640),
                                            (32, 576, 1536)])
def test_merge_widths(n_h, d_ck, d_c, B, n_splits):
    r, d_h, stride = 4, 128, 700
    seqs = [690 - 71 * b for b in range(B)]
    rng = np.random.default_rng(d_c + B + n_splits)
    idx = synth.draw_elite_idx(rng, n_h, d_h, r)
    dk, dv = (d_ck, d_c - d_ck) if d_ck else (d_c, d_c)
    _, _, W_uk, _ = synth.draw_weights(rng, 64, n_h, d_h, r, dk)
    _, _, _, W_uv = synth.draw_weights(rng, 64, n_h, d_h, r, dv)
    ke64, c64 = synth.draw_cache_planes(rng, B * stride, n_h, r, d_c)
    q = synth.draw_query(rng, B, n_h, d_h)
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "bf16", 10000.0)
    ke, c, qd, Wukd, Wuvd = (dev(a, "bf16") for a in (ke64, c64, q, W_uk, W_uv))
    pos = np.array(seqs) - 1
    args = (qd, i32(pos), i32(seqs), max(seqs), stride, Wukd, Wuvd, i32(idx), ke, c, n_splits)
    out = gpu_slrd_decode(dims, d_ck, *args) if d_ck else gpu_decode(dims, *args)
    keh, ch = host64(ke).reshape(B, stride, n_h, -1), host64(c).reshape(B, stride, -1)
    rest = (seqs, host64(Wukd), host64(Wuvd), idx, d_h, 10000.0)
    ref = (orc.slrd_decode_attn(host64(qd), pos, keh, ch[..., :dk], ch[..., dk:], *rest) if d_ck
           else orc.decode_attn(host64(qd), pos, keh, ch, *rest))
    assert orc.max_abs_rel(host64(out), ref) <= TOL["bf16"]


def _equal_weights(n_h, d_ck, d_c, B, columns):
    """A call whose queries are zero over three splits of 16 rows, a tile each: every row counts the same, so the merged latent of column j
    is the mean of columns[j]'s three values.  W_uv has ones for these columns and zeros for the others."""
    r, d_h, S = 4, 128, 48
    dk, dv = (d_ck, d_c - d_ck) if d_ck else (d_c, d_c)
    c = torch.zeros(B, S, d_c)
    W_uv = torch.zeros(dv, n_h, d_h)
    for j, values in enumerate(columns):
        c[:, :, d_c - dv + j] = torch.tensor(values).repeat_interleave(16)
        W_uv[j] = 1
    z = lambda *size: torch.zeros(*size, dtype=torch.bfloat16, device=DEV)
    idx = i32(np.tile(np.arange(r), (n_h, 1)))
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "bf16", 10000.0)
    args = (z(B, n_h, d_h), i32([S - 1] * B), i32([S] * B), S, S, z(dk, n_h, d_h - 2 * r), W_uv.bfloat16().to(DEV), idx,
            z(B * S, n_h, 2 * r), c.bfloat16().reshape(B * S, d_c).to(DEV))
    return lambda ns: host64(gpu_slrd_decode(dims, d_ck, *args, ns) if d_ck else gpu_decode(dims, *args, ns))


# the separated values of an odd width, a single row of a width of neither chunk, a width of whole chunks whose rows have more
# splits than the LDS holds weights
FULL_WIDTH = [(32, 320, 640, 2, 3), (40, 448, 896, 33, 3), (32, 320, 640, 1, 3), (32, 0, 256, 9, 1024), (8, 192, 384, 1, 3)]


@pytest.mark.parametrize("n_h, d_ck, d_c, B, n_splits", FULL_WIDTH)
def test_merged_latent_is_multiplied_in_full(n_h, d_ck, d_c, B, n_splits):
    """Two columns whose merged values cancel but for 2^-13 / 3.  Sixteen bits of them would be wrong by 2^-17 or so, a
    sixteenth of that; fp32 products and sums by at most 2^-22 (sixteen roundings of 2^-26), the bf16 result by 2^-9 of it."""
    out = _equal_weights(n_h, d_ck, d_c, B, [(1.0, 2.0 ** -6, 2.0 ** -13), (-1.0, -2.0 ** -6, 0.0)])(n_splits)
    want = 2.0 ** -13 / 3
    assert np.max(np.abs(out - want)) <= 2.0 ** -22 + 2.0 ** -9 * want


@pytest.mark.parametrize("n_h, d_ck, d_c, B, n_splits", [f for f in FULL_WIDTH if f[1]])
def test_infinite_values_stay_infinite(n_h, d_ck, d_c, B, n_splits):
    out = _equal_weights(n_h, d_ck, d_c, B, [(1.0, float("inf"), 2.0)])(n_splits)
    assert np.all(out == np.inf)
