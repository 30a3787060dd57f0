"""The search's round kernel at the edges of its tiles (16 tokens, blocks of 32 queries, pieces of key tiles), and samples
too long for the kept residuals, against the float64 oracle: every choice an arg-min of the oracle's distances for the
GPU's own earlier choices, every reported distance the oracle's, to 2e-4 (fp32 sums of up to 10^7 terms) and the rounding of
the residuals."""
import numpy as np
import pytest

import paper_2503_01586_amd as ekv
from oracle import elitekv_oracle as orc
from test_gpu_search import RTOL, gpu_search

pytestmark = pytest.mark.gpu


def residual_rounding(q, k, h):
    """What rounding can make of a distance that vanishes (the last chunk leaves nothing): a pair's residual is a sum of d_h / 2
    chunks of two scores each, the vectors rotated and rounded before, every operation to 2^-24 of the terms so far."""
    T, _, d_h = q.shape
    size = lambda v: np.linalg.norm(v[:, h].reshape(T, d_h // 2, 2), axis=2)     # [T, chunks]
    terms = 2.0 * d_h ** -0.5 * float(np.sum(size(q) * np.cumsum(size(k), axis=0)))
    return (d_h // 2 + 16) * 2.0 ** -24 * terms


@pytest.mark.parametrize("T,n_h,d_h,r", [
    (1, 3, 16, 2), (16, 5, 8, 4), (17, 1, 128, 3), (33, 2, 66, 5), (48, 7, 16, 8), (129, 1, 64, 32), (530, 1, 16, 3),
    (395, 64, 16, 3),        # pieces of sixteen key tiles, residuals kept over three rounds
    (97, 2, 32, 8), (128, 8, 16, 4), (208, 3, 16, 2),        # few work-groups
    (97, 64, 8, 3), (128, 64, 6, 2), (208, 40, 8, 2),        # blocks of 64 x 64: the fewest tiles, whole blocks, thirteen tiles
    (145, 32, 6, 2),                                         # ... a block for each compute unit at most
    (225, 1, 128, 20), (257, 8, 16, 8),                      # ... residuals summed afresh in late rounds, one tile in the last row
    (1281, 2, 8, 2), (1408, 36, 4, 2),                       # ... many blocks, more than the cache holds (one work-group per item)
    (4097, 1, 4, 2),         # longer than what keeps the residuals; one token in the last tile
])
def test_search_at_tile_edges(T, n_h, d_h, r):
    rng = np.random.default_rng(T + d_h)
    mag = np.exp(rng.normal(0.0, 0.7, size=(1, n_h, d_h // 2))).repeat(2, axis=2)
    pos = np.sort(rng.choice(3 * T, size=T, replace=False))
    q, k = rng.standard_normal((T, n_h, d_h)) * mag, rng.standard_normal((T, n_h, d_h)) * mag
    last = (T - 1) // 16 * 16                    # a lost last tile would show in every distance
    q[last:] *= 8.0
    k[last:] *= 8.0
    q64, k64, elite, dist = gpu_search(q, k, pos, r, 10000.0)
    for h in range(n_h):
        assert len(set(elite[h].tolist())) == r and elite[h].min() >= 0 and elite[h].max() < d_h // 2
        floor = residual_rounding(q64, k64, h)
        for i in range(r):
            ref = orc.ropelite_distances(q64, k64, pos, elite[h, :i], h, d_h, 10000.0)
            c = int(elite[h, i])
            assert ref[c] <= float(np.min(ref)) * (1 + RTOL) + floor, (h, i)
            assert abs(dist[h, i] - ref[c]) <= RTOL * ref[c] + floor, (h, i)


@pytest.mark.parametrize("T,n_h,d_h,r", [(16, 5, 8, 4), (129, 1, 64, 32), (300, 8, 128, 8), (2048, 1, 16, 2)])
def test_search_in_the_least_workspace(T, n_h, d_h, r):
    """Without room for the residuals (here: the room of a longer sample that keeps none) they are summed again in every
    round: the same choices, the same distances to rounding."""
    rng = np.random.default_rng(T + d_h)
    mag = np.exp(rng.normal(0.0, 0.7, size=(1, n_h, d_h // 2))).repeat(2, axis=2)
    q, k, pos = (rng.standard_normal((T, n_h, d_h)) * mag, rng.standard_normal((T, n_h, d_h)) * mag, np.arange(T))
    _, _, elite, dist = gpu_search(q, k, pos, r, 10000.0)
    least = ekv.elitekv_ropelite_search_min_workspace_bytes(T, n_h, d_h, r)
    assert least < ekv.elitekv_ropelite_search_workspace_bytes(T, n_h, d_h, r)
    _, _, elite_least, dist_least = gpu_search(q, k, pos, r, 10000.0, ws_bytes=least)
    assert np.array_equal(elite, elite_least)
    assert np.max(np.abs(dist - dist_least)) <= RTOL * np.max(dist)
