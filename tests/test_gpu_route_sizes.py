"""The router at the sizes where its kernels change shape, against the oracle: a tile that spans more tables than it
stages, table searches of one, two and three rounds, and the number of tile counts up to which every scatter block
sums them itself (tiles x (buckets + 3) <= 6144) with one more and one fewer tile."""
import numpy as np
import pytest
import torch

import oracle
from helpers import random_placement

pytestmark = pytest.mark.gpu

TILE = 2048


@pytest.fixture(scope="module")
def G():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


@pytest.mark.parametrize("T,B,n,U,W", [
    (1, 3, 1, 1, 1), (64, 1, 700, 8, 8), (65, 2, 5000, 8, 4), (130, 1, 2048, 24, 8), (4097, 1, 3000, 8, 2),
    (5000, 2, 9000, 64, 8),
    (3, 7, 91 * TILE, 64, 8), (3, 7, 91 * TILE + 1, 64, 8),         # 91 x 67 = 6097 counts; one tile more: 6164
    (2, 5, TILE, 4096, 64), (2, 5, TILE + 1, 4096, 64),             # 4099 counts; 8198
    (2, 5, 23 * TILE - 5, 257, 257),                                # two buckets to a thread, 23 x 260 = 5980
])
def test_route_shapes(G, T, B, n, U, W):
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(T * 7 + n + U)
    cuts = np.sort(rng.integers(0, n + 1, T * B - 1)) if T * B > 1 else np.zeros(0, np.int64)
    offsets = np.concatenate([[0], cuts, [n]]).astype(np.int64)
    E = 37
    ids = rng.integers(0, E, n).astype(np.int64)
    row_base = (np.arange(T + 1) * E).astype(np.int64)
    placement = random_placement(rng, T * E, U, W)
    self_ = int(rng.integers(0, U))
    rc, st, bo, rows, pos, tc = G.hip_route(G.to_dev(ids), G.to_dev(offsets), T, B, G.to_dev(row_base),
                                            G.placement_dev(placement), U, W, self_, n=n)
    orc, ost, obo, orows, opos, otc = oracle.route_bucketize(ids, offsets, T, B, row_base, placement, U, W, self_, n=n)
    assert (rc, st) == (orc, ost) == (0, 0)
    assert np.array_equal(bo.cpu().numpy(), obo) and np.array_equal(tc.cpu().numpy(), otc)
    assert np.array_equal(rows.cpu().numpy(), orows) and np.array_equal(pos.cpu().numpy(), opos)
