"""The tiled fp32 kernels (the fp32 dtype, and bf16 widths the bf16 kernels are not compiled for) at the edges of their
tiles, against the float64 oracle.  Bounds: 1e-5 (fp32), 2e-2 (bf16), max-abs-rel."""
import numpy as np
import pytest
import torch

import elitekv_synth as synth
import paper_2503_01586_amd as ekv
from gpu_util import DEV, TOL, dev, gpu_append, gpu_decode, host64, i32, i64
from oracle import elitekv_oracle as orc

pytestmark = pytest.mark.gpu

# name: (d_model, n_heads, head_dim, r, d_ck (0 = joint), d_c, dtype, seq_len per row)
# blocks of 16 latent columns over eight waves: 1, 17 and 128 blocks; heads beside a group of 16; elite rows of none, one
# and many 16-byte pieces; sequences at the edges of a tile of 16; more splits than tiles
CASES = {
    "one_block": (64, 3, 32, 2, 0, 16, "fp32", [1, 15, 16, 17, 0]),
    "seventeen_blocks_17_heads": (100, 17, 64, 0, 0, 272, "fp32", [33, 5]),
    "widest_r64": (32, 16, 256, 64, 0, 2048, "fp32", [40]),
    "all_elite": (92, 8, 32, 16, 0, 48, "fp32", [50, 7, 129]),
    "7b": (128, 32, 128, 8, 0, 1536, "fp32", [100, 1]),
    "13b": (128, 40, 128, 8, 0, 1920, "fp32", [70]),
    "separated": (64, 5, 64, 4, 16, 144, "fp32", [0, 64, 65, 3, 100]),
    "separated_wide_values": (84, 32, 128, 8, 1024, 1536, "fp32", [37]),
    "bf16_320": (64, 8, 64, 4, 0, 320, "bf16", [33, 50, 200]),
    "bf16_13b_separated": (64, 40, 128, 8, 960, 1920, "bf16", [49]),
}


def _draw(name):
    d, n_h, d_h, r, d_ck, d_c, dt, lens = CASES[name]
    rng = np.random.default_rng(synth.SEED_BASE + 700 + len(name))
    idx = synth.draw_elite_idx(rng, n_h, d_h, r)
    dk, dv = (d_ck, d_c - d_ck) if d_ck else (d_c, d_c)
    n = lambda *s, std=1.0: rng.standard_normal(s) * std
    B, stride = len(lens), max(lens) + 3
    p = dict(W_ke=n(d, n_h, 2 * r, std=d ** -0.5), W_d=n(d, dk, std=d ** -0.5), W_d2=n(d, dv, std=d ** -0.5),
             W_uk=n(dk, n_h, d_h - 2 * r, std=dk ** -0.5), W_uv=n(dv, n_h, d_h, std=dv ** -0.5),
             ke=n(B * stride, n_h, 2 * r), c=n(B * stride, d_c), q=n(B, n_h, d_h))
    return rng, idx, stride, {k: dev(v, dt) for k, v in p.items()}


@pytest.mark.parametrize("name", list(CASES))
def test_tiled_decode_matches_oracle(name):
    d, n_h, d_h, r, d_ck, d_c, dt, lens = CASES[name]
    dims = ekv.make_dims(d, n_h, d_h, r, d_c, dt)
    assert ekv.elitekv_decode_path(dims, d_ck) == ekv.PATH_GENERIC
    rng, idx, stride, t = _draw(name)
    B, S = len(lens), max(lens)
    # whatever lies beyond a sequence's end must not matter
    for b, s in enumerate(lens):
        t["ke"][b * stride + s:(b + 1) * stride] = float("nan")
        t["c"][b * stride + s:(b + 1) * stride] = float("nan")
    h = {k: host64(v) for k, v in t.items()}
    q_pos = np.array([max(s - 1, 0) for s in lens])
    ke, c = h["ke"].reshape(B, stride, n_h, 2 * r), h["c"].reshape(B, stride, d_c)
    if d_ck:
        ref = orc.slrd_decode_attn(h["q"], q_pos, ke, c[:, :, :d_ck], c[:, :, d_ck:], lens, h["W_uk"], h["W_uv"], idx, d_h, 10000.0)
    else:
        ref = orc.decode_attn(h["q"], q_pos, ke, c, lens, h["W_uk"], h["W_uv"], idx, d_h, 10000.0)
    for ns in (0, 1, 2, 11):
        if d_ck:
            out = torch.full((B, n_h, d_h), float("nan"), dtype=t["q"].dtype, device=DEV)
            ws = torch.full((ekv.elitekv_slrd_decode_workspace_bytes(dims, d_ck, B, S, ns),), 0xFF, dtype=torch.uint8, device=DEV)
            ekv.elitekv_slrd_decode_attn(dims, d_ck, t["q"], i32(q_pos), i32(lens), S, stride, t["W_uk"], t["W_uv"], i32(idx),
                                         t["ke"], t["c"], out, ws, n_splits=ns)
            torch.cuda.synchronize()
        else:
            out = gpu_decode(dims, t["q"], i32(q_pos), i32(lens), S, stride, t["W_uk"], t["W_uv"], i32(idx), t["ke"], t["c"],
                             n_splits=ns)
        assert orc.max_abs_rel(host64(out), ref) <= TOL[dt], ns


# the merge reads ahead in batches of 64 splits for up to 512 work-groups (272 columns: two a head), and not for more; empty
# splits leave the workspace as it was (filled with NaN)
@pytest.mark.parametrize("B", [1, 64, 65])
@pytest.mark.parametrize("ns", [3, 63, 64, 65, 300])
def test_merge_of_few_and_many_rows(B, ns):
    n_h, d_h, r, d_c, S = 4, 32, 2, 272, 90
    dims = ekv.make_dims(64, n_h, d_h, r, d_c, "fp32")
    rng = np.random.default_rng(synth.SEED_BASE + 760 + ns)
    idx = synth.draw_elite_idx(rng, n_h, d_h, r)
    n = lambda *s, std=1.0: dev(rng.standard_normal(s) * std, "fp32")
    q, W_uk, W_uv = n(B, n_h, d_h), n(d_c, n_h, d_h - 2 * r, std=d_c ** -0.5), n(d_c, n_h, d_h, std=d_c ** -0.5)
    ke, c = n(B * S, n_h, 2 * r), n(B * S, d_c)
    lens = np.array([S] + [int(v) for v in rng.integers(0, S + 1, B - 1)])
    q_pos = np.maximum(lens - 1, 0)
    out = torch.full((B, n_h, d_h), float("nan"), device=DEV)
    ws = torch.full((ekv.elitekv_decode_workspace_bytes(dims, B, S, ns),), 0xFF, dtype=torch.uint8, device=DEV)
    ekv.elitekv_decode_attn(dims, q, i32(q_pos), i32(lens), S, S, W_uk, W_uv, i32(idx), ke, c, out, ws, n_splits=ns)
    torch.cuda.synchronize()
    ref = orc.decode_attn(host64(q), q_pos, host64(ke).reshape(B, S, n_h, 2 * r), host64(c).reshape(B, S, d_c), lens,
                          host64(W_uk), host64(W_uv), idx, d_h, 10000.0)
    assert orc.max_abs_rel(host64(out), ref) <= TOL["fp32"]


@pytest.mark.parametrize("name", ["one_block", "seventeen_blocks_17_heads", "all_elite", "7b", "separated",
                                  "separated_wide_values"])
@pytest.mark.parametrize("T", [1, 2, 3, 5, 9, 257])     # token tiles of 1, 2, 4 and 8; the serial kernel beyond 256
def test_tiled_append_matches_oracle(name, T):
    d, n_h, d_h, r, d_ck, d_c, dt, _ = CASES[name]
    dims = ekv.make_dims(d, n_h, d_h, r, d_c, dt)
    tiled = T <= 256 and 2 * r * n_h % 16 == 0          # whole slices of 16 columns; the others take the serial kernel
    assert ekv.elitekv_append_gemm_tile(dims, T, d_ck) == (ekv.TILE_FP32 if tiled else ekv.TILE_NONE)
    rng, idx, _, t = _draw(name)
    x, pos = dev(rng.standard_normal((T, d)), dt), rng.integers(0, 5000, T)
    slot = rng.permutation(T + 4)[:T]
    slot[T // 2] = -1                                    # skipped
    ke = torch.full((T + 4, n_h, 2 * r), 7.0, dtype=x.dtype, device=DEV)
    c = torch.full((T + 4, d_c), 7.0, dtype=x.dtype, device=DEV)
    h = {k: host64(v) for k, v in t.items()}
    if d_ck:
        ekv.elitekv_slrd_append(dims, d_ck, x, i32(pos), i64(slot), t["W_ke"], t["W_d"], t["W_d2"], i32(idx), ke, c)
        ke_r, ck_r, cv_r = orc.slrd_append(host64(x), pos, h["W_ke"], h["W_d"], h["W_d2"], idx, d_h, 10000.0)
        c_r = np.concatenate([ck_r, cv_r], axis=1)
    else:
        gpu_append(dims, x, i32(pos), i64(slot), t["W_ke"], t["W_d"], i32(idx), T + 4, ke, c)
        ke_r, c_r = orc.append(host64(x), pos, h["W_ke"], h["W_d"], idx, d_h, 10000.0)
    torch.cuda.synchronize()
    keep = slot >= 0
    assert orc.max_abs_rel(host64(c)[slot[keep]], c_r[keep]) <= TOL[dt]
    if r:
        assert orc.max_abs_rel(host64(ke)[slot[keep]], ke_r[keep]) <= TOL[dt]
    untouched = np.setdiff1d(np.arange(T + 4), slot[keep])
    assert np.all(host64(c)[untouched] == 7.0) and np.all(host64(ke)[untouched] == 7.0)


def test_scratch_limit_takes_the_plan_that_fits():
    """elitekv_decode_attn_noalloc: where the tiled plan is larger than the scratch and the any-shape plan is not, the call
    runs the latter and is not refused."""
    dims = ekv.make_dims(64, 32, 128, 2, 2048, "fp32")
    fits = lambda S: ekv.elitekv_decode_workspace_bytes(dims, 1, S, 0) <= ekv.NOALLOC_SCRATCH_BYTES
    S = next(s for s in range(64, 4096, 16) if not fits(s))
    rng = np.random.default_rng(3)
    idx = synth.draw_elite_idx(rng, 32, 128, 2)
    n = lambda *s, std=1.0: dev(rng.standard_normal(s) * std, "fp32")
    q, W_uk, W_uv = n(1, 32, 128), n(2048, 32, 124, std=2048 ** -0.5), n(2048, 32, 128, std=2048 ** -0.5)
    ke, c = n(S, 32, 4), n(S, 2048)
    out = torch.full((1, 32, 128), float("nan"), device=DEV)
    ekv.elitekv_decode_attn_noalloc(dims, q, i32([S - 1]), i32([S]), S, S, W_uk, W_uv, i32(idx), ke, c, out)
    torch.cuda.synchronize()
    ref = orc.decode_attn(host64(q), [S - 1], host64(ke)[None], host64(c)[None], [S], host64(W_uk), host64(W_uv), idx, 128,
                          10000.0)
    assert orc.max_abs_rel(host64(out), ref) <= TOL["fp32"]


@pytest.mark.parametrize("B", [1, 2, 3, 5, 8, 9])           # front launches of 1, 2, 4 and 8 rows; two launches beyond 8
@pytest.mark.parametrize("name", ["seventeen_blocks_17_heads", "all_elite", "7b"])
def test_tiled_step_matches_oracle(name, B):
    d, n_h, d_h, r, _, d_c, dt, _ = CASES[name]
    dims = ekv.make_dims(d, n_h, d_h, r, d_c, dt)
    rng, idx, _, t = _draw(name)
    lens = [1 + (37 * b) % 50 for b in range(B)]
    S, stride = max(lens), max(lens) + 2
    n = lambda *s: dev(rng.standard_normal(s), dt)
    x, q, ke, c = n(B, d), n(B, n_h, d_h), n(B * stride, n_h, 2 * r), n(B * stride, d_c)
    pos, slot = np.array(lens) - 1, np.arange(B) * stride + np.array(lens) - 1
    h = {k: host64(v) for k, v in t.items()}
    ke_r, c_r = orc.append(host64(x), pos, h["W_ke"], h["W_d"], idx, d_h, 10000.0)
    ke_all, c_all = host64(ke), host64(c)
    ke_all[slot], c_all[slot] = ke_r, c_r
    ref = orc.decode_attn(host64(q), pos, ke_all.reshape(B, stride, n_h, 2 * r), c_all.reshape(B, stride, d_c), lens, h["W_uk"],
                          h["W_uv"], idx, d_h, 10000.0)
    out = torch.full((B, n_h, d_h), float("nan"), dtype=x.dtype, device=DEV)
    ws = torch.full((ekv.elitekv_decode_step_workspace_bytes(dims, B, S),), 0xFF, dtype=torch.uint8, device=DEV)
    ke[i64(slot)], c[i64(slot)] = float("nan"), float("nan")        # the step writes the new rows before it reads them
    ekv.elitekv_decode_step(dims, x, q, i32(pos), i64(slot), i32(lens), S, stride, t["W_ke"], t["W_d"], t["W_uk"], t["W_uv"],
                            i32(idx), ke, c, out, ws)
    torch.cuda.synchronize()
    assert orc.max_abs_rel(host64(c), c_all) <= TOL[dt] and (r == 0 or orc.max_abs_rel(host64(ke), ke_all) <= TOL[dt])
    assert orc.max_abs_rel(host64(out), ref) <= TOL[dt]


@pytest.mark.parametrize("n_splits", [0, 126])
def test_scratch_limit_keeps_the_kernels(n_splits):
    """... and with the same number of splits its result is elitekv_decode_attn's bit for bit.  126 is the largest count whose
    partials the scratch holds (qe 512 + q~ 262144 + 126 x 262400 bytes), without room for the merged latents; at
    2048 tokens the automatic count is 128."""
    dims = ekv.make_dims(64, 32, 128, 2, 2048, "fp32")
    B, S, stride = 1, 2048, 2049
    assert ekv.elitekv_decode_workspace_bytes(dims, B, S, n_splits) > ekv.NOALLOC_SCRATCH_BYTES
    rng = np.random.default_rng(4)
    idx = synth.draw_elite_idx(rng, 32, 128, 2)
    n = lambda *s, std=1.0: dev(rng.standard_normal(s) * std, "fp32")
    q, W_uk, W_uv = n(B, 32, 128), n(2048, 32, 124, std=2048 ** -0.5), n(2048, 32, 128, std=2048 ** -0.5)
    ke, c = n(stride, 32, 4), n(stride, 2048)
    out = torch.full((B, 32, 128), float("nan"), device=DEV)
    ekv.elitekv_decode_attn_noalloc(dims, q, i32([S - 1]), i32([S]), S, stride, W_uk, W_uv, i32(idx), ke, c, out,
                                    n_splits=n_splits)
    torch.cuda.synchronize()
    same = gpu_decode(dims, q, i32([S - 1]), i32([S]), S, stride, W_uk, W_uv, i32(idx), ke, c, n_splits=126)
    assert torch.equal(out, same)


@pytest.mark.parametrize("n_splits", [1, 3])
def test_a_tile_of_keys_at_minus_infinity(n_splits):
    """Elite keys of -inf hide their tokens: whole tiles of them (16 tokens, the first of every split) leave the others'
    softmax as it is."""
    d_h, n_h, d_c, S, hidden = 32, 16, 48, 150, 60
    dims = ekv.make_dims(64, n_h, d_h, 2, d_c, "fp32")
    rng = np.random.default_rng(6)
    idx = synth.draw_elite_idx(rng, n_h, d_h, 2)
    n = lambda *s, std=1.0: dev(rng.standard_normal(s) * std, "fp32")
    q, W_uk, W_uv = n(1, n_h, d_h), n(d_c, n_h, d_h - 4, std=d_c ** -0.5), n(d_c, n_h, d_h, std=d_c ** -0.5)
    ke, c = n(S, n_h, 4), n(S, d_c)
    for h in range(n_h):                                     # at position 0 the query enters as it is: make it positive
        q[0, h, 2 * int(idx[h, 0])] = 1.0
    ke[:hidden, :, 0] = float("-inf")
    out = gpu_decode(dims, q, i32([0]), i32([S]), S, S, W_uk, W_uv, i32(idx), ke, c, n_splits=n_splits)
    ref = orc.decode_attn(host64(q), [0], host64(ke)[None, hidden:], host64(c)[None, hidden:], [S - hidden], host64(W_uk),
                          host64(W_uv), idx, d_h, 10000.0)
    assert orc.max_abs_rel(host64(out), ref) <= TOL["fp32"]
