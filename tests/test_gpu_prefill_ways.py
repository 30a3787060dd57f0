"""Every way a prefill's flash attention goes (elitekv_prefill_plan: pairs of blocks two work-groups to a compute unit, 128- and
256-query blocks, each whole or divided among work-groups), for both elite widths, against the float64 oracle on sampled queries
and the absorbed form on every query.  The plan of each case is asserted, so that a change of the rule moves no case unnoticed.

rising: the latent rows are multiples of one direction, growing along the sequence, so a head's scores rise for some queries and
fall for others by far more than the kernels' slack: running maxima are raised over live accumulators, and pieces of a divided
block have maxima that differ by as much."""
import numpy as np
import pytest
import torch

import elitekv_synth as synth
import paper_2503_01586_amd as ekv
from oracle import elitekv_oracle as orc

from gpu_util import DEV, TOL, dev, host64, i32
from test_gpu_parity import _draw, shape

D_C = 256
# way, heads, r, rows per sequence, T, kinds
WAYS = [
    (ekv.PREFILL_PAIRS, 32, 8, [124, 70], 64, "causal random"),
    (ekv.PREFILL_PAIRS, 32, 4, [200], 200, "causal rising"),
    (ekv.PREFILL_PAIRS, 32, 8, [300 - 11 * b for b in range(9)], 160, "causal"),          # pairs of blocks
    (ekv.PREFILL_PAIRS, 32, 4, [500, 390, 301, 400, 260, 490, 300, 400], 260, "random rising"),   # an unpaired middle one
    (ekv.PREFILL_128, 8, 8, [300, 191], 150, "causal random"),
    (ekv.PREFILL_128, 32, 4, [700], 640, "causal rising"),
    (ekv.PREFILL_256, 32, 8, [500, 311, 257], 257, "random rising"),
    (ekv.PREFILL_256, 32, 4, [301, 500, 420], 300, "causal rising"),
    (ekv.PREFILL_128_DIVIDED, 8, 8, [1500], 64, "causal rising"),
    (ekv.PREFILL_128_DIVIDED, 16, 4, [1500, 700], 100, "random rising"),
    (ekv.PREFILL_256_DIVIDED, 40, 8, [3000, 2500], 400, "random rising"),
    (ekv.PREFILL_256_DIVIDED, 48, 4, [6500], 1000, "rising"),
]
CASES = [(*w[:5], kind) for w in WAYS for kind in w[5].split()]


def _dims(n_h, r):
    return ekv.make_dims(64, n_h, 128, r, D_C, "bf16", 10000.0)


def _ws_bytes(dims, B, T, S):
    """Room for divided blocks whatever the size function asks for."""
    return ekv.elitekv_prefill_attn_workspace_bytes(dims, B, T, S) + (80 << 20)


def _plan(n_h, r, rows, T):
    dims = _dims(n_h, r)
    return ekv.elitekv_prefill_plan(dims, len(rows), T, max(rows), _ws_bytes(dims, len(rows), T, max(rows)))


@pytest.mark.parametrize("way, n_h, r, rows, T, kinds", WAYS)
def test_the_way_of_a_case(way, n_h, r, rows, T, kinds):
    assert _plan(n_h, r, rows, T) == way


@pytest.mark.gpu
@pytest.mark.parametrize("way, n_h, r, rows, T, kind", CASES)
def test_every_way_matches(way, n_h, r, rows, T, kind):
    assert _plan(n_h, r, rows, T) == way
    B, S = len(rows), max(rows)
    stride = S + 3
    sh = shape(64, n_h, 128, r, D_C, "bf16")
    rng, idx, _, _, W_uk, W_uv, _, _ = _draw(sh, 1, 1, 900 + T + r)
    ke64, c64 = synth.draw_cache_planes(rng, B * stride, n_h, r, D_C)
    if kind == "rising":
        at = np.tile(np.arange(stride) / S, B)
        c64 = 0.05 * c64 + (15.0 * at + 0.3 * np.sin(np.arange(B * stride)))[:, None] * rng.standard_normal(D_C)[None]
    if kind == "random":
        kv_len = np.stack([rng.integers(0, n + 1, size=T) for n in rows])
        kv_len[:, ::17] = 0
        kv_len[:, 5] = np.array(rows)
    else:
        kv_len = np.array([[max(n - T + t + 1, 0) for t in range(T)] for n in rows])
    q_pos = np.maximum(kv_len - 1, 0)
    dims = _dims(n_h, r)
    ked, cd, qd, Wukd, Wuvd = (dev(a, "bf16") for a in (ke64, c64, rng.standard_normal((B, T, n_h, 128)), W_uk, W_uv))
    out, other = (torch.full((B, T, n_h, 128), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.full((_ws_bytes(dims, B, T, S),), 0xFF, dtype=torch.uint8, device=DEV)
    args = (dims, qd, i32(q_pos.reshape(-1)), i32(kv_len.reshape(-1)), S, stride, Wukd, Wuvd, i32(idx), ked, cd)
    ekv.elitekv_prefill_attn(*args, out, ws)
    torch.cuda.synchronize()
    o = host64(out)
    assert np.all(np.isfinite(o)) and np.all(o[kv_len == 0] == 0.0)
    pick = sorted({0, 5, T // 2, T - 1, min(127, T - 1), min(255, T - 1)} | set(int(t) for t in rng.choice(T, size=3)))
    pick = pick if S < 2000 else pick[::2] + [T - 1]
    ref = orc.multiquery_attn(host64(qd)[:, pick], q_pos[:, pick], host64(ked).reshape(B, stride, n_h, -1),
                              host64(cd).reshape(B, stride, -1), kv_len[:, pick], host64(Wukd), host64(Wuvd), idx, 128, 10000.0)
    assert orc.max_abs_rel(o[:, pick], ref) <= TOL["bf16"]
    ws2 = torch.empty(ekv.elitekv_multiquery_workspace_bytes(dims, B, T, S), dtype=torch.uint8, device=DEV)
    ekv.elitekv_multiquery_attn(*args, other, ws2)
    torch.cuda.synchronize()
    # two bf16 computations of the same quantity, each within the bound of the exact result
    assert np.max(np.abs(o - host64(other))) <= 2 * TOL["bf16"] * np.max(np.abs(o))


@pytest.mark.gpu
@pytest.mark.parametrize("n_h, rows, T, way", [(8, [1500, 900], 64, ekv.PREFILL_128_DIVIDED), (40, [3000], 1000, ekv.PREFILL_256_DIVIDED)])
def test_divided_blocks_replay_from_a_graph(n_h, rows, T, way):
    """The arrival counts are cleared by a launch of the call itself: every replay finds whatever the workspace holds."""
    B, S, r = len(rows), max(rows), 8
    dims = _dims(n_h, r)
    assert _plan(n_h, r, rows, T) == way
    rng = np.random.default_rng(3)
    ke64, c64 = synth.draw_cache_planes(rng, B * S, n_h, r, D_C)
    _, _, W_uk, W_uv = synth.draw_weights(rng, 64, n_h, 128, r, D_C)
    ked, cd, Wukd, Wuvd, qd = (dev(a, "bf16") for a in (ke64, c64, W_uk, W_uv, rng.standard_normal((B, T, n_h, 128))))
    idx = i32(synth.draw_elite_idx(rng, n_h, 128, r))
    q_pos = i32(np.concatenate([np.arange(n - T, n) for n in rows]))
    kv_len = q_pos + 1
    out = torch.zeros(B, T, n_h, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.full((_ws_bytes(dims, B, T, S),), 0xFF, dtype=torch.uint8, device=DEV)

    def call(stream):
        ekv.elitekv_prefill_attn(dims, qd, q_pos, kv_len, S, S, Wukd, Wuvd, idx, ked, cd, out, ws, stream=stream)

    call(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    want = out.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        call(side.cuda_stream)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call(torch.cuda.current_stream().cuda_stream)
    for rep in range(4):
        out.fill_(float("nan"))
        ws.fill_(0xFF if rep % 2 else 0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), "replay %d differs from the eager call" % rep
        call(torch.cuda.current_stream().cuda_stream)          # the program's own calls in between
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("dims5, B, T, S, way", [
    ((4096, 32, 128, 8, 1536), 1, 64, 128, ekv.PREFILL_PAIRS), ((4096, 32, 128, 8, 1536), 8, 512, 512, ekv.PREFILL_PAIRS),
    ((4096, 32, 128, 8, 1536), 16, 700, 700, ekv.PREFILL_PAIRS), ((4096, 32, 128, 4, 768), 32, 300, 600, ekv.PREFILL_PAIRS),
    ((5120, 40, 128, 8, 1920), 8, 1024, 1024, ekv.PREFILL_PAIRS), ((4096, 32, 128, 8, 1536), 1, 2048, 2048, ekv.PREFILL_128),
    ((4096, 32, 128, 8, 1536), 2, 2048, 2048, ekv.PREFILL_256), ((4096, 32, 128, 8, 1536), 1, 128, 8000, ekv.PREFILL_128_DIVIDED),
    ((5120, 40, 128, 8, 1920), 2, 1021, 8000, ekv.PREFILL_256_DIVIDED)])
def test_what_was_measured_as_the_faster_way(dims5, B, T, S, way):
    """Short prompts and batches of them: two work-groups to a compute unit; long ones: one."""
    dims = ekv.make_dims(*dims5, "bf16")
    assert ekv.elitekv_prefill_plan(dims, B, T, S, 1 << 40) == way


@pytest.mark.parametrize("d_c, d_ck", [(64, 0), (96, 32), (160, 0), (160, 96), (256, 224), (320, 160), (1536, 0), (1536, 576)])
@pytest.mark.parametrize("n_h, r", [(8, 8), (16, 4), (40, 8)])
def test_the_rebuild_clears_the_arrival_counts(n_h, r, d_c, d_ck):
    """Divided blocks count arrivals in memory that the rebuild's GEMM clears; its staged tiles do not."""
    dims = ekv.make_dims(64, n_h, 128, r, d_c, "bf16")
    for S in (513, 1500, 8000):
        for T in (64, 500):
            if ekv.elitekv_prefill_plan(dims, 1, T, S, 1 << 40, d_ck) != ekv.PREFILL_ABSORBED:
                assert ekv.elitekv_prefill_gemm_tile(dims, T, S, d_ck) not in (ekv.TILE_NONE, ekv.TILE_STAGED_64_128,
                                                                              ekv.TILE_STAGED_256_128)
