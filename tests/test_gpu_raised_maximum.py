"""Split attention whose scores rise and fall from tile to tile by more than the slack of the running maximum (2^8), so that it
is raised over live accumulators: every kernel whose lanes form the probabilities of the scores they finalised, against the
float64 oracle.  The latents lean towards the absorbed queries of all heads by an amount that changes from tile to tile: the
logits are that amount plus a unit normal, and the rounding of the absorbed query (2^-9 of every term, of independent signs)
stays below 2^-9 * 20 / sqrt(d_c / 3) of a logit, far inside the parity bound of bf16."""
import numpy as np
import pytest
import torch

import elitekv_synth as synth
import paper_2503_01586_amd as ekv
from oracle import elitekv_oracle as orc

from gpu_util import DEV, TOL, dev, gpu_decode, host64, i32
from test_gpu_slrd import gpu_slrd_decode

pytestmark = pytest.mark.gpu

LEAN = np.array([0.0, 9.0, 2.0, 16.0, 16.0, 5.0, 20.0, 1.0, 11.0])   # natural logits, tile by tile


def leaning_latents(rng, c, q, W_uk, idx):
    """c [rows, d_c] leaned towards the absorbed query of every head (q [n_h, d_h])."""
    n_h, d_h = q.shape
    qt = np.zeros((n_h, c.shape[1]))
    for h in range(n_h):
        chunks = set(idx[h].tolist())
        others = [i for i in range(d_h) if i // 2 not in chunks]
        qt[h] = W_uk[:, h] @ q[h, others] / np.sqrt(d_h)
    u = (qt / np.sum(qt * qt, axis=1, keepdims=True)).sum(axis=0)
    return c + LEAN[np.arange(c.shape[0]) // 16 % len(LEAN)][:, None] * u[None]


@pytest.mark.parametrize("n_h,r,d_c,T", [
    (32, 8, 128, 1),       # two waves
    (32, 4, 768, 1),       # four waves, two work-groups per compute unit
    (40, 8, 1920, 1),      # head-group pairs, one wave per SIMD
    (32, 8, 2048, 1), (32, 16, 1536, 1),
    (32, 8, 1536, 3), (32, 8, 1024, 4),      # several queries
])
@pytest.mark.parametrize("n_splits", [1, 2])
def test_scores_that_rise_and_fall(n_h, r, d_c, T, n_splits):
    rng = np.random.default_rng(d_c + n_h + T)
    d_h, lens = 128, [145, 17, 112, 33]
    B, stride = len(lens), max(lens) + 3
    idx = synth.draw_elite_idx(rng, n_h, d_h, r)
    _, _, W_uk, W_uv = synth.draw_weights(rng, 64, n_h, d_h, r, d_c)
    ke64, c64 = synth.draw_cache_planes(rng, B * stride, n_h, r, d_c)
    q = np.repeat(synth.draw_query(rng, B, n_h, d_h)[:, None], T, axis=1)
    c64 = np.concatenate([leaning_latents(rng, c64[b * stride:(b + 1) * stride], q[b, 0], W_uk, idx) for b in range(B)])
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "bf16", 10000.0)
    ked, cd, qd, Wukd, Wuvd = (dev(a, "bf16") for a in (ke64, c64, q, W_uk, W_uv))
    seen = np.array([[n - (T - 1 - t) for t in range(T)] for n in lens])
    pos = seen - 1
    ke_h, c_h = host64(ked).reshape(B, stride, n_h, -1), host64(cd).reshape(B, stride, -1)
    if T == 1:
        out = host64(gpu_decode(dims, qd[:, 0].contiguous(), i32(pos[:, 0]), i32(lens), max(lens), stride, Wukd, Wuvd, i32(idx),
                                ked, cd, n_splits=n_splits))
        ref = orc.decode_attn(host64(qd)[:, 0], pos[:, 0], ke_h, c_h, lens, host64(Wukd), host64(Wuvd), idx, d_h, 10000.0)
    else:
        o = torch.full((B, T, n_h, d_h), float("nan"), dtype=torch.bfloat16, device=DEV)
        ws = torch.full((ekv.elitekv_multiquery_workspace_bytes(dims, B, T, max(lens), n_splits),), 0xFF, dtype=torch.uint8, device=DEV)
        ekv.elitekv_multiquery_attn(dims, qd, i32(pos.reshape(-1)), i32(seen.reshape(-1)), max(lens), stride, Wukd, Wuvd, i32(idx),
                                    ked, cd, o, ws, n_splits=n_splits)
        torch.cuda.synchronize()
        out = host64(o)
        ref = orc.multiquery_attn(host64(qd), pos, ke_h, c_h, seen, host64(Wukd), host64(Wuvd), idx, d_h, 10000.0)
    assert np.all(np.isfinite(out))
    assert orc.max_abs_rel(out, ref) <= TOL["bf16"]


def latents_leaning_to_thirds(rng, c, q, W_uk, idx):
    """The same towards another third of the heads in every tile."""
    tile = np.arange(c.shape[0]) // 16
    out = c.copy()
    for k in range(3):
        out[tile % 3 == k] = leaning_latents(rng, c, q[k::3], W_uk[:, k::3], idx[k::3])[tile % 3 == k]
    return out


@pytest.mark.parametrize("n_h,r,d_c,d_ck,T", [
    (32, 8, 128, 0, 1), (40, 8, 1920, 0, 1), (32, 4, 768, 0, 1), (32, 8, 1536, 0, 1),
    (32, 8, 1536, 0, 3), (40, 8, 1920, 0, 3),
    # separated latents: the waves of the values finalise scores too, from the partial scores of the others alone
    (32, 8, 128, 64, 1), (32, 8, 768, 384, 1), (32, 16, 1536, 576, 1), (32, 8, 1536, 576, 1),
    (32, 8, 1536, 576, 3), (32, 4, 768, 192, 4),
])
@pytest.mark.parametrize("n_splits", [1, 2])
def test_heads_that_rise_in_different_tiles(n_h, r, d_c, d_ck, T, n_splits):
    """In every tile some heads raise their maximum and the others keep theirs, over the accumulators of both."""
    rng = np.random.default_rng(d_c + d_ck + n_h + T)
    d_h, lens = 128, [145, 17, 112, 33]
    B, stride, dk = len(lens), max(lens) + 3, d_ck or d_c
    idx = synth.draw_elite_idx(rng, n_h, d_h, r)
    _, _, W_uk, _ = synth.draw_weights(rng, 64, n_h, d_h, r, dk)
    _, _, _, W_uv = synth.draw_weights(rng, 64, n_h, d_h, r, d_c - d_ck)
    ke64, c64 = synth.draw_cache_planes(rng, B * stride, n_h, r, d_c)
    q = np.repeat(synth.draw_query(rng, B, n_h, d_h)[:, None], T, axis=1)
    for b in range(B):
        rows = slice(b * stride, (b + 1) * stride)
        c64[rows, :dk] = latents_leaning_to_thirds(rng, c64[rows, :dk], q[b, 0], W_uk, idx)
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "bf16", 10000.0)
    assert ekv.elitekv_decode_path(dims, d_ck) == 1
    ked, cd, qd, Wukd, Wuvd = (dev(a, "bf16") for a in (ke64, c64, q, W_uk, W_uv))
    seen = np.array([[n - (T - 1 - t) for t in range(T)] for n in lens])
    pos = seen - 1
    ke_h, c_h = host64(ked).reshape(B, stride, n_h, -1), host64(cd).reshape(B, stride, -1)
    o = torch.full((B, T, n_h, d_h), float("nan"), dtype=torch.bfloat16, device=DEV)
    sep = (d_ck,) if d_ck else ()
    size = ekv.elitekv_slrd_multiquery_workspace_bytes if d_ck else ekv.elitekv_multiquery_workspace_bytes
    attend = ekv.elitekv_slrd_multiquery_attn if d_ck else ekv.elitekv_multiquery_attn
    ws = torch.full((size(dims, *sep, B, T, max(lens), n_splits),), 0xFF, dtype=torch.uint8, device=DEV)
    attend(dims, *sep, qd, i32(pos.reshape(-1)), i32(seen.reshape(-1)), max(lens), stride, Wukd, Wuvd, i32(idx), ked, cd, o, ws,
           n_splits=n_splits)
    torch.cuda.synchronize()
    if d_ck:
        ref = orc.slrd_multiquery_attn(host64(qd), pos, ke_h, c_h[..., :dk], c_h[..., dk:], seen, host64(Wukd), host64(Wuvd), idx, d_h,
                                       10000.0)
    else:
        ref = orc.multiquery_attn(host64(qd), pos, ke_h, c_h, seen, host64(Wukd), host64(Wuvd), idx, d_h, 10000.0)
    assert np.all(np.isfinite(host64(o)))
    assert orc.max_abs_rel(host64(o), ref) <= TOL["bf16"]


@pytest.mark.parametrize("r,d_c,d_ck", [(8, 128, 64), (8, 768, 384), (16, 1536, 576), (8, 1536, 576)])
@pytest.mark.parametrize("exponent", [-120, -127])
def test_probability_below_the_normal_range(r, d_c, d_ck, exponent):
    """A row whose probability is 2^exponent and whose values are 2^(-1 - exponent) adds a half to every column of the merged latent,
    also where the probability is a subnormal number.  Its logit lies 88 below the largest: the rounding of the absorbed query (2^-9
    of every one of d_ck terms, of independent signs) moves it by 88 * 2^-9 / sqrt(d_ck / 3) < 0.04, and its half by that share."""
    rng = np.random.default_rng(d_c)
    n_h, d_h, S = 32, 128, 20
    idx = np.repeat(synth.draw_elite_idx(rng, 1, d_h, r), n_h, axis=0)
    W_uk = np.repeat(synth.draw_weights(rng, 64, 1, d_h, r, d_ck)[2], n_h, axis=1)
    W_uv = synth.draw_weights(rng, 64, n_h, d_h, r, d_c - d_ck)[3]
    q = np.repeat(synth.draw_query(rng, 1, 1, d_h), n_h, axis=1)
    others = [i for i in range(d_h) if i // 2 not in set(idx[0].tolist())]
    qt = W_uk[:, 0] @ q[0, 0, others] / np.sqrt(d_h)
    logit = np.full(S, -300.0)
    logit[0], logit[1] = 0.0, exponent * np.log(2.0)
    ke, c = np.zeros((S, n_h, 2 * r)), np.empty((S, d_c))
    c[:, :d_ck] = logit[:, None] * (qt / np.sum(qt * qt))[None]
    c[:, d_ck:] = rng.standard_normal((S, d_c - d_ck))
    c[1, d_ck:] = 2.0 ** (-1 - exponent)
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "bf16", 10000.0)
    ked, cd, qd, Wukd, Wuvd = (dev(a, "bf16") for a in (ke, c, q, W_uk, W_uv))
    out = host64(gpu_slrd_decode(dims, d_ck, qd, i32([S - 1]), i32([S]), S, S, Wukd, Wuvd, i32(idx), ked, cd, 1))
    ch = host64(cd).reshape(1, S, -1)
    ref = orc.slrd_decode_attn(host64(qd), [S - 1], host64(ked).reshape(1, S, n_h, -1), ch[..., :d_ck], ch[..., d_ck:], [S], host64(Wukd),
                               host64(Wuvd), idx, d_h, 10000.0)
    assert orc.max_abs_rel(out, ref) <= TOL["bf16"] + 0.04
