"""The sort and the planner's selection at the sizes where their kernels change shape, against the oracle: 1024-pair
and 4096-pair tiles, the largest numbers of tiles whose counts the scatter sums itself, the passes of the selection's
sort that are left out where the counts are small, and the compaction with and without a scan of its own."""
import numpy as np
import pytest
import torch

import oracle
from helpers import entry

pytestmark = pytest.mark.gpu

S, TAG, Z = oracle.PLAN_SELECT, oracle.PLAN_TAG, oracle.PLAN_ALLOW_ZERO
TILE = 8192                                          # rows of one compaction tile


@pytest.fixture(scope="module")
def G():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


@pytest.mark.parametrize("m", [1, 1023, 1024, 1025, 65536, 65537, 262144, 262145])
@pytest.mark.parametrize("R", [3, 200, 1 << 10, (1 << 17) + 1, 1 << 20, 3_000_000])
def test_sort_sizes(G, m, R):
    check_sort(G, m, R)


@pytest.mark.parametrize("m", [512 * 4096, 512 * 4096 + 1, 1024 * 4096, 1024 * 4096 + 1])
@pytest.mark.parametrize("R", [200, 3_000_000, 1 << 30])
def test_sort_sizes_with_a_scan(G, m, R):
    """Up to 512 tiles the scan's chunks are of 32 tiles, then of 64; up to 16 chunks, 1024 tiles, the scatter adds up
    their sums, beyond them a launch of its own does."""
    check_sort(G, m, R)


def check_sort(G, m, R):
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(m + R)
    rows = np.where(rng.random(m) < 0.5, rng.integers(0, min(R, 7), m), rng.integers(0, R, m)).astype(np.int64)
    rows[0] = R - 1
    pos = np.arange(m, dtype=np.int32)
    srows = torch.full((m,), -7, dtype=torch.int32, device=G.DEV)
    spos = torch.full((m,), -7, dtype=torch.int32, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_sort_lookups(G.to_dev(rows), G.to_dev(pos), 0, m, R, m, srows, spos, st)
    orc, ost, osr, osp = oracle.sort_lookups(rows, pos, 0, m, R, m)
    assert orc == 0 and int(st.item()) == ost == 0
    assert np.array_equal(srows.cpu().numpy().view(np.uint32), osr)
    assert np.array_equal(spos.cpu().numpy().view(np.uint32), osp)


@pytest.mark.parametrize("m", [128 * 4096 + 1, 384 * 4096, 384 * 4096 + 1, 2048 * 4096 + 4095, (1 << 25) - 1, 1 << 25])
@pytest.mark.parametrize("R", [200, 700_000, (1 << 32) - 2])
def test_sort_group_sizes(G, m, R):
    """A scan thread takes up to 4, 12 or 32 groups of tiles, a group one tile, two or three (more than 1024, 2048 tiles),
    and from 2^25 pairs on keys and values lie apart between passes; one to four passes.  Against torch's stable sort."""
    import paper_2301_02959_amd as fs
    torch.manual_seed(m % 1000)
    rows = torch.randint(0, R, (m,), device=G.DEV)
    rows[torch.rand(m, device=G.DEV) < 0.3] = R - 1                            # a popular row
    pos = torch.arange(m, dtype=torch.int32, device=G.DEV)
    srows = torch.full((m,), -7, dtype=torch.int32, device=G.DEV)
    spos = torch.full((m,), -7, dtype=torch.int32, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_sort_lookups(rows, pos, 0, m, R, m, srows, spos, st)
    want, order = torch.sort(rows, stable=True)
    assert int(st.item()) == 0
    assert torch.equal(srows.long() & 0xFFFFFFFF, want)
    assert torch.equal(spos.long(), order)


@pytest.mark.parametrize("R", [1, 1024, 128 * 1024, 128 * 1024 + 1, 64 * 4096, 64 * 4096 + 1, 1024 * TILE, 1024 * TILE + 1])
@pytest.mark.parametrize("bits,share", [(1, 0.9), (10, 0.01), (11, 0.3), (20, 0.05), (21, 0.3), (30, 0.1), (31, 0.3), (32, 0.02)])
def test_selection_sizes(G, R, bits, share):
    """Counts of up to `bits` bits on `share` of the rows: passes are left out at 10, 20 and 26 bits."""
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(R + bits)
    counts = np.where(rng.random(R) < share, 1 + rng.geometric(0.4, R), 0).astype(np.uint64)
    some = rng.integers(0, R, 50)
    counts[some] = rng.integers(1, 1 << bits, 50)
    counts = np.minimum(counts, (1 << bits) - 1)
    counts[some[0]] = 1 << (bits - 1)
    counts = counts.astype(np.uint32)
    for flags, budget in [(S | TAG, max(1, R // 50)), (S | Z, R)]:
        if R > 1_000_000 and flags & Z:
            continue
        placement = np.full(R, entry(2, 3), np.uint32)
        oc, opl = counts.copy(), placement.copy()
        orc, ost, osel = oracle.plan_replication(None, None, 1, 1, None, R, oc, flags, budget, 1, opl, n=0)
        dev = torch.from_numpy(counts.view(np.int32).copy()).to(G.DEV)
        pl = G.placement_dev(placement)
        sel = torch.full((budget,), -7, dtype=torch.int64, device=G.DEV)
        num = torch.full((1,), -7, dtype=torch.int64, device=G.DEV)
        fs.fs_plan_replication(None, None, 1, 1, None, 0, R, dev, flags, budget, 1, sel, num, pl)
        assert orc == ost == 0 and int(num.item()) == len(osel)
        assert np.array_equal(sel[:len(osel)].cpu().numpy(), osel)
        assert np.array_equal(pl.cpu().numpy().view(np.uint32), opl if flags & TAG else placement)
    # the tier planner reads the same sorted counts, keys included
    params = dict(num_samples=1000, B=64, U=8, W=4, dp_multiplier=6, granule=8, a2a_global=1, a2a_intra=6, ar_global=3, ar_cross=2)
    cuts = torch.zeros(fs.FS_TIER_CUTS, dtype=torch.int64, device=G.DEV)
    rows = torch.full((R,), -7, dtype=torch.int64, device=G.DEV)
    fs.fs_plan_tiers(torch.from_numpy(counts.view(np.int32).copy()).to(G.DEV), R, params, 3, rows, R, cuts)
    orc, ocuts, orows = oracle.plan_tiers(counts, params, 3)
    assert orc == 0 and cuts.cpu().numpy().tolist() == ocuts.tolist()
    assert np.array_equal(rows[:len(orows)].cpu().numpy(), orows)


@pytest.mark.parametrize("R", [1000, 100_000, 300_000, 1 << 26, (1 << 26) + 1])
def test_selection_at_every_number_of_passes(G, R):
    """Largest counts on both sides of every digit's end: 10, 20 and 26 bits up to 2^26 rows, 8, 16 and 24 beyond.  The order
    is that of numpy's stable sort of the candidates."""
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(R)
    K = min(R // 3, 60_000)
    rows = np.sort(rng.choice(R, K, replace=False))
    dev = torch.zeros(R, dtype=torch.int32, device=G.DEV)
    sel = torch.zeros(K, dtype=torch.int64, device=G.DEV)
    num = torch.zeros(1, dtype=torch.int64, device=G.DEV)
    cuts = torch.zeros(fs.FS_TIER_CUTS, dtype=torch.int64, device=G.DEV)
    params = dict(num_samples=1000, B=64, U=8, W=4, dp_multiplier=6, granule=8, a2a_global=1, a2a_intra=6, ar_global=3, ar_cross=2)
    at = G.to_dev(rows)
    for bits in [1, 8, 9, 10, 11, 16, 17, 20, 21, 24, 25, 26, 27, 32]:
        counts = 1 + rng.integers(0, 1 << rng.integers(0, bits, K), K).astype(np.uint64)     # every length up to `bits`
        counts = np.minimum(counts, (1 << bits) - 1)
        counts[rng.integers(0, K)] = 1 << (bits - 1)
        dev[at] = G.to_dev(counts.astype(np.uint32).view(np.int32))
        order = rows[np.argsort(-counts.astype(np.int64), kind="stable")]
        fs.fs_plan_replication(None, None, 1, 1, None, 0, R, dev, S, K, 1, sel, num)
        assert int(num.item()) == K and np.array_equal(sel.cpu().numpy(), order), bits
        sel.fill_(-7)
        fs.fs_plan_tiers(dev, R, params, 3, sel, K, cuts)
        n = int(cuts[fs.FS_CUT_N_DP] + cuts[fs.FS_CUT_N_FLEX])
        assert int(cuts[fs.FS_CUT_CANDIDATES]) == K and int(cuts[fs.FS_CUT_SUM_ALL]) == int(counts.sum()), bits
        assert np.array_equal(sel[:n].cpu().numpy(), order[:n]), bits


@pytest.mark.parametrize("tiles", [1025, 2048, 2049, 15 * 1024, 15 * 1024 + 1])
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("zero", [False, True])
def test_compaction_tiles(G, tiles, off, zero):
    """Numbers of compaction tiles around the runs of the scan in LDS (odd lengths, at most 15) and beyond it, the last
    tile ragged; counters 16-byte aligned or not; dense stretches, full waves and empty ones."""
    import paper_2301_02959_amd as fs
    R = tiles * TILE - (777 if off else 0)
    if zero and tiles > 1025:
        pytest.skip("every row a candidate: the smallest size is enough")
    torch.manual_seed(tiles + off)
    buf = torch.zeros(R + off, dtype=torch.int32, device=G.DEV)
    counts = buf[off:]
    some = torch.randint(0, R, (30_000,), device=G.DEV)
    counts[some] = torch.randint(1, 300, (30_000,), dtype=torch.int32, device=G.DEV)
    for lo in (0, 3 * TILE, 5 * TILE + 2048, R - 5000):                         # whole waves of candidates, the ragged end
        counts[lo:lo + 2048] = 1
    counts[-1] = 70_000
    K = R if zero else int((counts > 0).sum())
    sel = torch.full((K,), -7, dtype=torch.int64, device=G.DEV)
    num = torch.zeros(1, dtype=torch.int64, device=G.DEV)
    fs.fs_plan_replication(None, None, 1, 1, None, 0, R, counts, S | (Z if zero else 0), K, 1, sel, num)
    rows = torch.arange(R, device=G.DEV) if zero else torch.nonzero(counts > 0).flatten()
    order = torch.sort(counts[rows], descending=True, stable=True)[1]
    assert int(num.item()) == K and torch.equal(sel, rows[order])


def sort_workspace_bytes(m, R):
    import ctypes
    import paper_2301_02959_amd as fs
    size = ctypes.c_size_t(0)
    assert fs._typed().fs_sort_lookups(None, None, 0, m, R, max(m, 1), None, None, None, ctypes.byref(size), None, None) == 0
    return size.value


def test_the_sorts_workspace():
    """What two passes ask for serves any number of rows and any smaller batch: a buffer for the pairs, 1024 counts of 4 bytes
    for 4096 of them, up to 5 MB; never more than a second buffer beyond it is asked for."""
    before = 0
    for m in (0, 1, 1000, 65_536, 65_537, 262_144, 262_145, 1_000_000, 4_194_304, 4_194_305, (1 << 25) - 1, 1 << 25, (1 << 31) - 1):
        need = sort_workspace_bytes(m, 200)
        assert before <= need <= 8 * m + m + (5 << 20)
        for R in (1, 1 << 10, 1 << 20, (1 << 20) + 1, 1 << 30, (1 << 32) - 2):
            second = R > 1 << 20 and m < 1 << 25
            assert need <= sort_workspace_bytes(m, R) <= need + (8 * m + 256 if second else 0)
        before = need


@pytest.mark.parametrize("R", [1000, 1 << 20, 80_000_000, (1 << 32) - 2])
@pytest.mark.parametrize("m", [1, 1025, 65_536, 65_537, 262_145, 1_100_000, 1 << 25])
def test_one_to_four_passes_in_that_workspace(G, R, m):
    """In what every R is served with, in what this one asks for and in one byte less than that; nothing is written past the
    end of the workspace or of the outputs."""
    import paper_2301_02959_amd as fs
    gen = torch.Generator(device=G.DEV).manual_seed(m)
    rows = torch.randint(0, R, (m,), device=G.DEV, generator=gen)
    rows[torch.rand(m, device=G.DEV, generator=gen) < 0.2] = R // 2
    pos = torch.arange(m, dtype=torch.int32, device=G.DEV)
    want, order = torch.sort(rows, stable=True)
    need, asked = sort_workspace_bytes(m, 200), sort_workspace_bytes(m, R)
    for size in sorted({need, max(need, asked - 1), asked}):
        guarded = torch.full((size + 4096,), 85, dtype=torch.uint8, device=G.DEV)
        out = torch.full((2 * m + 128,), -7, dtype=torch.int32, device=G.DEV)
        srows, spos = out[1:m + 1], out[m + 65:2 * m + 65]
        st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
        fs.fs_sort_lookups(rows, pos, 0, m, R, m, srows, spos, st, workspace=guarded[:size])
        assert int(st.item()) == 0 and torch.equal(srows.long() & 0xFFFFFFFF, want) and torch.equal(spos.long(), order)
        assert bool((guarded[size:] == 85).all())
        assert all(bool((part == -7).all()) for part in (out[:1], out[m + 1:m + 65], out[2 * m + 65:]))
    assert fs.fs_sort_lookups(rows, pos, 0, m, R, m, srows, spos, st, workspace=guarded[:need - 1], raise_on_error=False) == 5


def test_a_workspace_for_more_rows_serves_fewer():
    """The scratch size does not shrink as the rows grow, also where the sort goes over to larger tiles."""
    import ctypes
    import paper_2301_02959_amd as fs
    sizes = []
    for R in [1, 1024, 65536, 65537, 100_000, 131_072, 131_073, 150_000, 262_144, 262_145, 600_000, 1024 * TILE, 1024 * TILE + 1]:
        size = ctypes.c_size_t(0)
        assert fs.lib().fs_plan_replication(None, None, 1, 1, None, ctypes.c_int64(0), ctypes.c_int64(R), None, S, ctypes.c_int64(8),
                                            ctypes.c_int64(1), None, None, None, None, ctypes.byref(size), None, None) == 0
        sizes.append(size.value)
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("T,B,n", [(1, 1, 1), (1, 8, 2048), (3, 5, 2049), (2, 4096, 100_000), (8193, 1, 100_000), (70, 200, 524_289),
                                   (5, 3, 256 * 32768), (5, 3, 256 * 32768 + 1), (5, 300_000, 3_000_001)])
@pytest.mark.parametrize("bad", [False, True])
def test_histogram_sizes(G, T, B, n, bad):
    """The offsets checked by the counting blocks themselves or by blocks of their own, spans of every length below
    the longest; bad offsets (the last pair of them) count nothing either way."""
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(T + n)
    E = 4001
    offsets = np.concatenate([[0], np.sort(rng.integers(0, n + 1, T * B - 1)), [n]]).astype(np.int64)
    if bad:
        offsets[-2] = n + 1
        if T * B == 1:
            offsets[-1] = n + 1
    ids = np.where(rng.random(n) < 0.5, 7, rng.integers(0, E, n)).astype(np.int64)
    row_base = (np.arange(T + 1) * E).astype(np.int64)
    counts = rng.integers(0, 3, T * E).astype(np.uint32)
    dev = torch.from_numpy(counts.view(np.int32).copy()).to(G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_plan_replication(G.to_dev(ids), G.to_dev(offsets), T, B, G.to_dev(row_base), n, T * E, dev, fs.FS_PLAN_ACCUMULATE, dev_status=st)
    oc = counts.copy()
    orc, ost, _ = oracle.plan_replication(ids, offsets, T, B, row_base, T * E, oc, oracle.PLAN_ACCUMULATE, n=n)
    assert orc == 0 and int(st.item()) == ost and (ost != 0) == bad
    assert np.array_equal(dev.cpu().numpy().view(np.uint32), oc)


@pytest.mark.parametrize("n", [2048, 256 * 2048, 256 * 2048 + 1])
@pytest.mark.parametrize("law", ["one row", "all different", "64 rows"])
def test_histogram_tables(G, n, law):
    """The small table of spans of 2048 ids and the large one: counts that wrap their entry's 10 bits, every id another
    row, few rows that share slots."""
    import paper_2301_02959_amd as fs
    R = 300_000_000
    row = {"one row": torch.full((n,), R - 1, device=G.DEV), "all different": (torch.arange(n, device=G.DEV) * 571 + 5) % R,
           "64 rows": (torch.arange(n, device=G.DEV) % 64) * 4_194_301}[law]
    offsets, row_base = (torch.tensor([0, end], device=G.DEV) for end in (n, R))
    counts = torch.zeros(R, dtype=torch.int32, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_plan_replication(row, offsets, 1, 1, row_base, n, R, counts, fs.FS_PLAN_ACCUMULATE, dev_status=st)
    want_rows, want = torch.unique(row, return_counts=True)
    assert int(st.item()) == 0 and torch.equal(counts[want_rows].long(), want)
    assert int(counts.sum(dtype=torch.int64)) == n


@pytest.mark.parametrize("first", [16383, 16384, 16385, 20001, 32767])
def test_table_ends_inside_a_span(G, first):
    """A first table of rows that are all different fills a span's slots (32 k ids a span), then the rows are another table's:
    few popular ones, and, after as many ids again, a third table's."""
    import paper_2301_02959_amd as fs
    n, E = 8_400_000, 10_000_000
    ends = [first, first + (32768 - first) // 2, n]
    ids = torch.arange(n, device=G.DEV) * 7 % E
    ids[ends[0]:ends[1]] = 3
    ids[ends[1]:32768 * 2] %= 5
    offsets = torch.tensor([0, *ends], device=G.DEV)
    row_base = torch.tensor([0, E, 2 * E, 3 * E], device=G.DEV)
    counts = torch.zeros(3 * E, dtype=torch.int32, device=G.DEV)
    counts[E + 3] = -2                                     # 2^32 - 2: pinned at the maximum
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_plan_replication(ids, offsets, 3, 1, row_base, n, 3 * E, counts, fs.FS_PLAN_ACCUMULATE, dev_status=st)
    rows = ids.clone()
    rows[ends[0]:ends[1]] += E
    rows[ends[1]:] += 2 * E
    want = torch.bincount(rows, minlength=3 * E)
    if ends[1] - ends[0] > 1:
        want[E + 3] = 0xFFFFFFFF
        assert int(st.item()) == fs.FS_DEV_COUNT_OVERFLOW
    else:
        want[E + 3] += 0xFFFFFFFE
        assert int(st.item()) == 0
    assert torch.equal(counts.long() & 0xFFFFFFFF, want)


@pytest.mark.parametrize("held", [8191, 8192, 16383, 16384, 81920 - 32769, 81920 - 32768, 81920 - 2049, 81920 - 2048, 81920 - 2047])
def test_what_is_left_of_a_span_where_a_table_ends(G, held):
    """Spans of 80 k ids: after so many of them every other span goes on in another table, over an empty one between; ids of
    popular rows among ids that are all different."""
    import paper_2301_02959_amd as fs
    n, E, span = 40_000_000, 1_000_000, 81920
    ends = torch.arange(40, device=G.DEV) * 2 * span + held
    offsets = torch.cat([ends.new_zeros(1), ends.repeat_interleave(2), ends.new_tensor([n])])
    T = offsets.numel() - 1
    at = torch.arange(n, device=G.DEV)
    ids = at * 7919 % E
    ids[::3] %= 50
    row_base = torch.arange(T + 1, device=G.DEV) * E
    counts = torch.zeros(T * E, dtype=torch.int32, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_plan_replication(ids, offsets, T, 1, row_base, n, T * E, counts, fs.FS_PLAN_ACCUMULATE, dev_status=st)
    tables = torch.searchsorted(offsets[1:].contiguous(), at, right=True)
    assert int(st.item()) == 0 and torch.equal(counts.long(), torch.bincount(tables * E + ids, minlength=T * E))


@pytest.mark.parametrize("n", [2048, 256 * 2048, 256 * 2048 + 1, 256 * 2048 + 255, 256 * 2048 + 256, 700_001, 256 * 30_720 + 1, 256 * 32_768])
def test_batches_are_counted_in_one_launch(G, n):
    """Up to 256 spans the counting blocks check the offsets themselves, and shorter spans never make more of them."""
    import paper_2301_02959_amd as fs
    ids = torch.randint(0, 999, (n,), device=G.DEV)
    offsets, row_base = (torch.tensor([0, end], device=G.DEV) for end in (n, 999))
    counts = torch.zeros(999, dtype=torch.int32, device=G.DEV)
    fs.fs_prof_begin(16)
    fs.fs_plan_replication(ids, offsets, 1, 1, row_base, n, 999, counts, fs.FS_PLAN_ACCUMULATE)
    assert [name for name, _ in fs.fs_prof_end(16)] == ["plan_histogram"]
    assert torch.equal(counts.long(), torch.bincount(ids, minlength=999))
