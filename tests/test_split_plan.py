"""The automatic split count of the matrix-core decode path: no second round of work-groups for a few of them, no
more splits than tiles, never zero."""
import pytest

import paper_2503_01586_amd as ekv


@pytest.mark.parametrize("shape,slots_per_cu", [((4096, 32, 128, 8, 1536), 1), ((5120, 40, 128, 8, 1920), 1),
                                                ((4096, 32, 128, 4, 768), 2)])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 16, 20, 33, 64, 127, 128, 129, 255, 256, 257, 700])
@pytest.mark.parametrize("S", [1, 16, 17, 256, 5001, 32768])
def test_one_round_of_work_groups(shape, slots_per_cu, B, S):
    dims = ekv.make_dims(*shape, "bf16")
    ns = ekv.elitekv_decode_auto_splits(dims, B, S)
    groups, tiles = B * ((shape[1] + 31) // 32), (S + 15) // 16
    slots = 256 * (slots_per_cu if groups >= 16 else 1)
    assert 1 <= ns <= tiles
    assert ns == 1 or groups * ns <= slots or groups > slots // 2
    # as many splits as one round holds, or as few as give the same tiles per split
    most = min(tiles, max(1, slots // groups))
    assert -(-tiles // ns) <= -(-tiles // most)
