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


@pytest.mark.parametrize("T,B,n,U,W,slots", [
    (1, 1, 512, 2, 1, True), (2, 3, 513, 3, 3, False), (64, 2, 164 * 512, 64, 8, True), (5, 9, 164 * 512 + 1, 64, 8, False),
    (65, 3, 84 * 512 - 1, 128, 8, False), (4, 2, 84 * 512 + 511, 128, 8, True),          # 83 x 131 = 10873 counts of 512 lookups
    (3, 5, 512 * 512, 8, 8, False), (3, 5, 512 * 512 + 1, 8, 8, True), (2, 7, 512 * 1024, 8, 2, False), (1, 8, 512 * 1024 + 1, 8, 2, False),
    (4, 4, 500 * 1024, 64, 8, True), (4, 4, 500 * 1024 + 1, 64, 8, False),               # 500 x 67 = 33500 counts of 1024 lookups
    (2, 2, 255 * 1024, 128, 64, False), (2, 2, 255 * 1024 + 1, 128, 64, False), (64, 1, 3000, 129, 129, False),
])
def test_small_tiles(G, T, B, n, U, W, slots):
    """Tiles of 512 lookups up to 11000 counts, of 1024 up to 33500, at most 512 of them and up to 128 buckets; empty tables
    among 64 and more; with and without the replica slots."""
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(T + n + U)
    cuts = np.sort(rng.choice(rng.integers(0, n + 1, 5), T * B - 1)) if T * B > 1 else np.zeros(0, np.int64)   # most segments empty
    offsets = np.concatenate([[0], cuts, [n]]).astype(np.int64)
    E = 41
    ids = rng.integers(0, E, n).astype(np.int64)
    row_base = (np.arange(T + 1) * E).astype(np.int64)
    placement = random_placement(rng, T * E, U, W)
    self_ = int(rng.integers(0, U))
    args = (G.to_dev(ids), G.to_dev(offsets), T, B, G.to_dev(row_base), G.placement_dev(placement))
    rc, st, bo, rows, pos, tc = G.hip_route(*args, U, W, self_, n=n)
    orc, ost, obo, orows, opos, otc = oracle.route_bucketize(ids, offsets, T, B, row_base, placement, U, W, self_, n=n)
    assert (rc, st) == (orc, ost) == (0, 0)
    assert np.array_equal(bo.cpu().numpy(), obo) and np.array_equal(tc.cpu().numpy(), otc)
    assert np.array_equal(rows.cpu().numpy(), orows) and np.array_equal(pos.cpu().numpy(), opos)
    if slots:
        bo2, rows2, pos2 = torch.zeros_like(bo), torch.zeros_like(rows), torch.zeros_like(pos)
        out = torch.full((n,), -7, dtype=torch.int32, device=G.DEV)
        fs.fs_route_bucketize_slots(*args, n, U, W, self_, bo2, rows2, pos2, out)
        assert torch.equal(bo2, bo) and torch.equal(rows2, rows) and torch.equal(pos2, pos)
        entries = placement[orows]
        owner = (entries & 0x3FFFFFFF).astype(np.int64)
        assert np.array_equal(out.cpu().numpy(), np.where((entries >> 30 == 0) & (owner != 0x3FFFFFFF), owner, -1))


@pytest.mark.parametrize("U", [1, 8, 24, 64, 128, 129, 4096])
def test_a_workspace_for_more_lookups_serves_fewer(U):
    import paper_2301_02959_amd as fs
    edges = [k * step + d for step in (512, 1024, 2048) for k in (1, 64, 83, 84, 164, 165, 255, 256, 500, 501, 512) for d in (-1, 0, 1)]
    sizes = [fs.route_workspace_bytes(2, 3, n, U, 1, 0) for n in sorted(edges)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("U", [1, 254, 255, 256, 257, 4096])
@pytest.mark.parametrize("tiers", [True, False])
def test_an_empty_batch_of_many_buckets(G, U, tiers):
    import paper_2301_02959_amd as fs
    offsets, row_base = torch.zeros(7, dtype=torch.int64, device=G.DEV), torch.tensor([0, 4, 8], device=G.DEV)
    none64, none32 = torch.zeros(1, dtype=torch.int64, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV)
    buckets = torch.full((U + 3,), 77, dtype=torch.int64, device=G.DEV)
    counts = torch.full((4,), 77, dtype=torch.int64, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_route_bucketize(none64, offsets, 2, 3, row_base, torch.zeros(8, dtype=torch.int32, device=G.DEV), 0, U, 1, 0,
                          buckets[1:U + 2], none64, none32, counts[:3] if tiers else None, st)
    assert buckets.tolist() == [77] + [0] * (U + 1) + [77] and int(st.item()) == 0
    assert counts.tolist() == ([0, 0, 0, 77] if tiers else [77] * 4)


@pytest.mark.parametrize("n", [1, 512, 513, 2048, 40_000, 128 * 512, 255 * 1024, 512 * 512, 512 * 1024 + 1, 4_000_000])
def test_a_workspace_for_more_buckets_serves_fewer(n):
    import paper_2301_02959_amd as fs
    sizes = [fs.route_workspace_bytes(2, 3, n, U, 1, 0) for U in (1, 2, 8, 63, 64, 65, 82, 83, 127, 128, 129, 130, 200, 512, 4096)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("n", [256 * TILE, 256 * TILE + 1, 256 * TILE + 777])
@pytest.mark.parametrize("U,self_", [(1, 0), (2, 0), (2, 1), (3, 1), (64, 5)])
@pytest.mark.parametrize("owners", ["one", "tables", "hot"])
def test_where_most_lookups_go_to_one_other_bucket(G, n, U, self_, owners):
    """Every row on one other GPU, whole tables on one owner each, one hot row: the counts that the ballots take and
    those that are left to LDS adds, on either side of one tile for every CU."""
    rng = np.random.default_rng(n + U + len(owners))
    T, E = 3, 50
    offsets = np.array([0, n // 3, n // 2, n], np.int64)
    ids = np.where(rng.random(n) < (0.6 if owners == "hot" else 0.0), 7, rng.integers(0, E, n)).astype(np.int64)
    row_base = (np.arange(T + 1) * E).astype(np.int64)
    row = np.arange(T * E)
    owner = {"one": np.full(T * E, (self_ + 1) % U), "tables": (row // E + self_) % U, "hot": row % U}[owners]
    placement = ((2 << 30) | owner).astype(np.uint32)
    rc, st, bo, rows, pos, tc = G.hip_route(G.to_dev(ids), G.to_dev(offsets), T, 1, G.to_dev(row_base),
                                            G.placement_dev(placement), U, 1, self_, n=n)
    orc, ost, obo, orows, opos, otc = oracle.route_bucketize(ids, offsets, T, 1, row_base, placement, U, 1, self_, n=n)
    assert (rc, st) == (orc, ost) == (0, 0)
    assert np.array_equal(bo.cpu().numpy(), obo) and np.array_equal(tc.cpu().numpy(), otc)
    assert np.array_equal(rows.cpu().numpy(), orows) and np.array_equal(pos.cpu().numpy(), opos)


@pytest.mark.parametrize("U", [255, 256, 257, 300, 513, 1023, 1024, 1025, 1500, 2047, 2048, 2049, 4095, 4096])
def test_buckets_a_thread_holds_in_registers(G, U):
    """Buckets that do not share out evenly over a scatter block's 256 threads, with one tile more than the blocks sum
    themselves."""
    rng = np.random.default_rng(U)
    n = (6144 // (U + 3) + 1) * TILE - 11
    T, B, E = 2, 9, 3 * U
    offsets = np.concatenate([[0], np.sort(rng.integers(0, n + 1, T * B - 1)), [n]]).astype(np.int64)
    ids = rng.integers(0, E, n).astype(np.int64)
    row_base = (np.arange(T + 1) * E).astype(np.int64)
    placement = random_placement(rng, T * E, U, 1)
    self_ = U - 1
    rc, st, bo, rows, pos, tc = G.hip_route(G.to_dev(ids), G.to_dev(offsets), T, B, G.to_dev(row_base),
                                            G.placement_dev(placement), U, 1, self_, n=n)
    orc, ost, obo, orows, opos, otc = oracle.route_bucketize(ids, offsets, T, B, row_base, placement, U, 1, self_, n=n)
    assert (rc, st) == (orc, ost) == (0, 0)
    assert np.array_equal(bo.cpu().numpy(), obo) and np.array_equal(tc.cpu().numpy(), otc)
    assert np.array_equal(rows.cpu().numpy(), orows) and np.array_equal(pos.cpu().numpy(), opos)
