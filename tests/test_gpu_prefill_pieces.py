"""Query blocks whose key tiles are divided among several work-groups (few blocks over a long cache), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2503_01586_amd as ekv
from gpu_util import DEV, TOL, dims_of, host64, i32
from oracle import elitekv_oracle as orc
from test_gpu_parity import shape
from test_gpu_prefill import CASES, _run

pytestmark = pytest.mark.gpu

PIECES = {
    # one block per head, many pieces; a last tile that is not full
    "pieces_one_block": (shape(64, 8, 128, 8, 256, "bf16"), [3001], 64, "causal", 16),
    # sequences far shorter than the bound: pieces without a tile
    "pieces_short_sequences": (shape(64, 8, 128, 8, 256, "bf16"), [3000, 400, 100], 100, "causal", 12),
    # queries that see nothing of some pieces, or nothing at all
    "pieces_random": (shape(64, 8, 128, 4, 256, "bf16"), [2500], 300, "random", 24),
    # 256-query blocks, their last rows past the end, stretches over two heads
    "pieces_of_wide_blocks": (shape(64, 40, 128, 8, 256, "bf16"), [6500], 1000, "causal", 3),
}
CASES.update(PIECES)


@pytest.mark.parametrize("name", list(PIECES))
def test_divided_blocks_match_the_oracle(name):
    sh, rows, T, B, stride, rng, idx, qd, q_pos, kv_len, ked, cd, Wukd, Wuvd, dims, o, n_sample, S = _run(name)
    n_h, d_h = sh["n_heads"], sh["head_dim"]
    pick = sorted(set([0, T - 1, min(127, T - 1), min(255, T - 1)] + list(rng.choice(T, size=n_sample, replace=False))))
    ref = orc.multiquery_attn(host64(qd)[:, pick], q_pos[:, pick], np.nan_to_num(host64(ked)).reshape(B, stride, n_h, -1),
                              np.nan_to_num(host64(cd)).reshape(B, stride, -1), kv_len[:, pick], host64(Wukd), host64(Wuvd),
                              idx, d_h, sh["rope_base"])
    assert orc.max_abs_rel(o[:, pick], ref) <= TOL["bf16"]


def test_the_order_of_arrival_does_not_matter():
    a, b = (_run("pieces_one_block")[15] for _ in range(2))
    assert np.array_equal(a, b)


def test_planes_without_rows():
    """Nothing is rebuilt and nothing is seen: zero rows."""
    sh = shape(64, 8, 128, 8, 256, "bf16")
    dims, T, S = dims_of(sh), 300, 200
    z = lambda *size: torch.zeros(*size, dtype=torch.bfloat16, device=DEV)
    out = torch.full((1, T, 8, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ekv.elitekv_prefill_attn_workspace_bytes(dims, 1, T, S),), 0xFF, dtype=torch.uint8, device=DEV)
    idx = torch.arange(8, dtype=torch.int32, device=DEV).repeat(8, 1)
    ekv.elitekv_prefill_attn(dims, torch.randn(1, T, 8, 128, device=DEV).bfloat16(), i32(np.arange(T)), i32(np.arange(T)), S, S,
                             z(256, 8, 112), z(256, 8, 128), idx, z(1, 8, 16), z(1, 256), out, ws,
                             plane_rows=0)
    torch.cuda.synchronize()
    assert torch.count_nonzero(out) == 0 and not torch.isnan(out).any()


def test_a_workspace_of_the_rebuilt_rows_alone():
    """No room for the states of divided blocks: a work-group per block, the same result up to the order of the sums."""
    sh, rows, T, B, stride, rng, idx, qd, q_pos, kv_len, ked, cd, Wukd, Wuvd, dims, o, n_sample, S = _run("pieces_one_block")
    least = -(-B * S * sh["n_heads"] * (2 * 128 - 2 * sh["r"]) * 2 // 256) * 256
    assert ekv.elitekv_prefill_attn_workspace_bytes(dims, B, T, S) > least
    out = torch.full((B, T, sh["n_heads"], 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    call = lambda n: ekv.elitekv_prefill_attn(dims, qd, i32(q_pos.reshape(-1)), i32(kv_len.reshape(-1)), S, stride, Wukd, Wuvd,
                                              i32(idx), ked, cd, out, torch.full((n,), 0xFF, dtype=torch.uint8, device=DEV))
    with pytest.raises(ekv.EliteKVError):
        call(least - 1)
    call(least)
    torch.cuda.synchronize()
    # both round fp32 sums to bf16: 2^-8 of the value, and the probabilities' bf16 rounding under another maximum
    assert np.max(np.abs(host64(out) - o)) <= 2 * TOL["bf16"] * np.max(np.abs(o))
