"""The automatic split count of the matrix-core decode path: whole rounds of work-groups, no more splits than tiles, never
zero; the workspace it asks for."""
import pytest

import paper_2503_01586_amd as ekv


@pytest.mark.parametrize("shape,slots_per_cu", [((4096, 32, 128, 8, 1536), 1), ((5120, 40, 128, 8, 1920), 1),
                                                ((4096, 32, 128, 4, 768), 2)])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 16, 20, 33, 43, 64, 86, 127, 128, 129, 150, 180, 255, 256, 257, 700])
@pytest.mark.parametrize("S", [1, 16, 17, 256, 5001, 32768])
def test_whole_rounds_of_work_groups(shape, slots_per_cu, B, S):
    dims = ekv.make_dims(*shape, "bf16")
    ns = ekv.elitekv_decode_auto_splits(dims, B, S)
    groups, tiles = B * ((shape[1] + 31) // 32), (S + 15) // 16
    slots = 256 * (slots_per_cu if groups >= 16 else 1)
    assert 1 <= ns <= tiles
    # as many splits as one, two or three rounds hold, or as few as give the same tiles per split
    rounds = [min(tiles, max(1, k * slots // groups)) for k in (1, 2, 3)]
    assert -(-tiles // ns) in [-(-tiles // most) for most in rounds]
    if groups <= slots and S == 32768:
        # long sequences leave at most a quarter of the chip idle
        assert groups * ns >= 0.74 * slots * -(-groups * ns // slots)


# name: (d_model, n_heads, head_dim, r, d_c, dtype, d_ck of the separated forms)
FORMS = {"7b_25": (4096, 32, 128, 8, 1536, "bf16", 576), "13b_25": (5120, 40, 128, 8, 1920, "bf16", 960),
         "7b_12": (4096, 32, 128, 4, 768, "bf16", 384), "fp32": (4096, 32, 128, 8, 1536, "fp32", 576),
         "bf16_320": (512, 8, 64, 4, 320, "bf16", 160), "any_shape": (36, 5, 36, 3, 17, "fp32", 5), "one_head": (64, 1, 64, 4, 64, "fp32", 16)}


@pytest.mark.parametrize("name", list(FORMS))
@pytest.mark.parametrize("B", [1, 2, 3, 4, 7, 8, 16, 33, 43, 64])
def test_workspace_of_a_longer_bound_covers_every_shorter_one(name, B):
    """A serving loop allocates once for the longest sequence and passes the current bound: the automatic workspace never
    falls as max_seq_len grows."""
    *shape, dtype, d_ck = FORMS[name]
    dims = ekv.make_dims(*shape, dtype)
    sizes = {
        "decode": lambda S: ekv.elitekv_decode_workspace_bytes(dims, B, S),
        "step": lambda S: ekv.elitekv_decode_step_workspace_bytes(dims, B, S),
        "block": lambda S: ekv.elitekv_block_step_workspace_bytes(dims, B, S),
        "multiquery": lambda S: ekv.elitekv_multiquery_workspace_bytes(dims, B, 5, S),
        "prefill": lambda S: ekv.elitekv_prefill_attn_workspace_bytes(dims, B, 5, S),
        "slrd_decode": lambda S: ekv.elitekv_slrd_decode_workspace_bytes(dims, d_ck, B, S),
        "slrd_step": lambda S: ekv.elitekv_slrd_decode_step_workspace_bytes(dims, d_ck, B, S),
        "slrd_block": lambda S: ekv.elitekv_slrd_block_step_workspace_bytes(dims, d_ck, B, S),
        "slrd_multiquery": lambda S: ekv.elitekv_slrd_multiquery_workspace_bytes(dims, d_ck, B, 5, S),
    }
    lengths = sorted(set(range(0, 8300, 16)) | set(range(1, 8300, 16)) | {5001, 16384, 32768, 32769, 131072, 131073})
    for form, of in sizes.items():
        before = 0
        for S in lengths:
            now = of(S)
            assert now >= before, (form, S, before, now)
            before = now


@pytest.mark.parametrize("n_h,d_c,B,S,splits", [
    (1, 64, 128, 700, 8), (1, 16, 32, 3000, 32), (2, 64, 300, 100, 2),     # any-shape kernels: about 1024 work-groups
    (1, 64, 32, 700, 8), (2, 64, 128, 700, 2), (1, 144, 128, 700, 2),      # tiled: one round of 256
])
def test_one_or_two_narrow_heads(n_h, d_c, B, S, splits):
    """Long shares of one narrow head keep the any-shape fp32 kernels, which take more and shorter splits."""
    for dtype in ("fp32", "bf16"):
        assert ekv.elitekv_decode_auto_splits(ekv.make_dims(64, n_h, 64, 4, d_c, dtype), B, S) == splits


def test_two_wave_work_groups_run_in_pairs():
    """A 128-column latent's work-groups have two waves: a compute unit runs two of them, and 200 rows two splits."""
    assert ekv.elitekv_decode_auto_splits(ekv.make_dims(1024, 32, 128, 4, 128, "bf16"), 200, 500) == 2
    assert ekv.elitekv_decode_auto_splits(ekv.make_dims(1024, 32, 128, 8, 1536, "bf16"), 200, 500) == 1


@pytest.mark.parametrize("name", ["7b_25", "13b_25", "7b_12"])
def test_a_prefill_workspace_serves_every_shorter_chunk(name):
    """Sized for the longest chunk, or for more sequences, a workspace has room for the divided blocks of the shorter ones too:
    a call goes the same way in it as in one of its own size."""
    *shape, dtype, d_ck = FORMS[name]
    dims = ekv.make_dims(*shape, dtype)
    size = lambda B, T, S: ekv.elitekv_prefill_attn_workspace_bytes(dims, B, T, S)
    chunks, rows, batches = (48, 128, 300, 656, 1024, 1808, 2048), (65, 512, 513, 1400, 2048, 8000), (1, 2, 5, 16)
    for B in batches:
        for S in rows:
            for T in chunks:
                if T > S:
                    continue
                held = size(B, T, S)
                assert held >= size(B, T, S - 1 if S > 66 else S)
                for b in (b for b in batches if b <= B):
                    for t in (t for t in chunks if t <= T):
                        assert held >= size(b, t, S)
                        for s in (s for s in rows if t <= s <= S):
                            assert (ekv.elitekv_prefill_plan(dims, b, t, s, held) ==
                                    ekv.elitekv_prefill_plan(dims, b, t, s, 1 << 40)), (b, t, s, B, T, S)


@pytest.mark.parametrize("name", list(FORMS))
@pytest.mark.parametrize("S", [100, 1000, 4096, 32768])
def test_a_step_workspace_serves_fewer_sequences(name, S):
    """A batch shrinks while it is served: the step's and the block's workspace never fall as sequences are added."""
    *shape, dtype, d_ck = FORMS[name]
    dims = ekv.make_dims(*shape, dtype)
    sizes = {
        "step": lambda B: ekv.elitekv_decode_step_workspace_bytes(dims, B, S),
        "slrd_step": lambda B: ekv.elitekv_slrd_decode_step_workspace_bytes(dims, d_ck, B, S),
        "block": lambda B: ekv.elitekv_block_step_workspace_bytes(dims, B, S),
        "slrd_block": lambda B: ekv.elitekv_slrd_block_step_workspace_bytes(dims, d_ck, B, S),
    }
    for form, of in sizes.items():
        before = 0
        for B in range(1, 65):
            now = of(B)
            assert now >= before, (form, B, before, now)
            before = now


@pytest.mark.parametrize("name", list(FORMS))
def test_an_append_workspace_serves_fewer_tokens(name):
    """The last chunk of a prompt is short: what was allocated for whole ones is enough for it."""
    *shape, dtype, d_ck = FORMS[name]
    dims = ekv.make_dims(*shape, dtype)
    for of in (lambda T: ekv.elitekv_append_workspace_bytes(dims, T), lambda T: ekv.elitekv_slrd_append_workspace_bytes(dims, d_ck, T)):
        sizes = [of(T) for T in list(range(0, 70)) + [128, 300, 2048, 100000]]
        assert sizes == sorted(sizes)
