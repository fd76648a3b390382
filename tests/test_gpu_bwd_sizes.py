"""The backward where its segmented sum changes shape, bit for bit against the oracle: up to 1024 chunks of 256
lookups are summed a block at a time out of LDS in slabs of up to 16 row pieces, more are walked by a wave each with
4 bytes to a lane (rows of up to 256 bytes) or 8."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_bwd import _check, _np_grad

pytestmark = pytest.mark.gpu

CHUNK = 256


@pytest.fixture(scope="module")
def G():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


def lookups(rng, n, R):
    """Sorted-friendly rows: a head that spans chunks, a stretch of pairs, a cold tail; positions a permutation."""
    head = np.minimum(rng.pareto(0.9, n // 2).astype(np.int64), R - 1)
    rows_i = rng.permutation(np.concatenate([head, rng.integers(0, R, n - n // 2)]))
    order = np.argsort(rows_i % 3, kind="stable")
    return rows_i[order], order.astype(np.int32)


def check_atomic(G, grad_np, grad_t, rows, pos, R, dt):
    """Variant 1 where a gradient row is looked up many times over.  The terms of a row are then not independent, and
    the 2-norm that the other tests take does not bound an fp32 sum of them in another order; what does is
    k u sum |term|, k the additions that one result passes through: up to 256 in its chunk, one per chunk of its run."""
    m = len(rows)
    _, _, ou, _, og64, _ = oracle.seq_grad_bwd(grad_np, rows, pos, 0, m, R, dtype=G.oracle_dtype(dt))
    rc, st, u, g, _ = G.hip_bwd(grad_t.to(G.DEV), G.to_dev(rows, torch.int64), G.to_dev(pos), 0, m, R, 1)
    assert (rc, st) == (0, 0) and np.array_equal(u.cpu().numpy(), ou)
    inv = torch.from_numpy(np.searchsorted(ou, rows))
    total = torch.zeros(len(ou), grad_t.shape[1], dtype=torch.float64)
    total.index_add_(0, inv, grad_t.double().abs()[torch.from_numpy(pos).long()])
    k = CHUNK + np.ceil(np.bincount(inv.numpy(), minlength=len(ou)) / CHUNK) + 1
    assert np.all(np.abs(g.double().cpu().numpy() - og64) <= k[:, None] * 2.0 ** -24 * total.numpy())


@pytest.mark.parametrize("dt,D", [("f16", 8), ("f32", 20), ("bf16", 128), ("f16", 136), ("f32", 100), ("bf16", 520)])
@pytest.mark.parametrize("m", [1, CHUNK - 1, CHUNK, CHUNK + 1, 5 * CHUNK + 3])
def test_few_chunks(G, dt, D, m):
    rng = np.random.default_rng(D + m)
    R = 700
    rows, pos = lookups(rng, m, R)
    gnp, gt = _np_grad(rng.standard_normal((m, D)).astype(np.float32), dt)
    _check(G, gnp, gt, rows, pos, 0, m, R, dt)


@pytest.mark.parametrize("dt,D", [("f32", 4), ("f32", 60), ("f32", 64), ("f32", 100), ("f16", 8), ("bf16", 24), ("bf16", 128), ("f16", 136),
                                  ("f16", 264)])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 31, 32, 33, 64, 65])
def test_few_rows_in_a_chunk(G, dt, D, R):
    """Chunks of at most as many run pieces as fit side by side with one column to a lane (64 rows of one piece of f32
    down to two of 128 16-bit columns), and of one more."""
    rng = np.random.default_rng(D + R)
    m = 4 * CHUNK + 77
    rows = np.sort(np.concatenate([np.arange(R), rng.integers(0, R, CHUNK - R), np.full(m - CHUNK, R - 1)]))   # all in the first chunk
    pos = (np.arange(m) % 611).astype(np.int32)
    pos = pos[np.lexsort((pos, rows))]
    gnp, gt = _np_grad(rng.standard_normal((611, D)).astype(np.float32), dt)
    _check(G, gnp, gt, rows, pos, 0, m, R, dt, atomic_too=False)
    check_atomic(G, gnp, gt, rows, pos, R, dt)


@pytest.mark.parametrize("dt,D", [("f32", 4), ("bf16", 72), ("f16", 128), ("f32", 68), ("f16", 264)])
@pytest.mark.parametrize("m", [1024 * CHUNK, 1024 * CHUNK + 1])
def test_around_the_rule(G, dt, D, m):
    rng = np.random.default_rng(D + m)
    R, n = 90_000, 3_000                             # few gradient rows, each used by many lookups
    rows, order = lookups(rng, m, R)
    pos = (np.arange(m) // (m // n + 1)).astype(np.int32)          # ascending
    gnp, gt = _np_grad(rng.standard_normal((n, D)).astype(np.float32), dt)
    _check(G, gnp, gt, rows, pos, 0, m, R, dt, atomic_too=False)
    check_atomic(G, gnp, gt, rows, pos, R, dt)


@pytest.mark.parametrize("m", [64 * CHUNK - 1, 64 * CHUNK, 64 * CHUNK + 1, 128 * CHUNK, 128 * CHUNK + 1])
def test_around_the_blocks_of_the_run_counts(G, m):
    """64 chunks are one block of the run counts, which then writes the totals itself; 65 are two and a scan."""
    rng = np.random.default_rng(m)
    rows, pos = lookups(rng, m, 9_000)
    gnp, gt = _np_grad(rng.standard_normal((m, 16)).astype(np.float32), "bf16")
    _check(G, gnp, gt, rows, pos, 0, m, 9_000, "bf16")


@pytest.mark.parametrize("R", [1, 2, 3])
@pytest.mark.parametrize("m", [1025 * CHUNK, 1025 * CHUNK + 77])
def test_walks_of_whole_chunks(G, R, m):
    """Every chunk one run that goes on into the next, the last chunk whole or ragged."""
    rng = np.random.default_rng(m + R)
    rows = np.sort(rng.integers(0, R, m))
    pos = (np.arange(m) % 911).astype(np.int32)
    pos = pos[np.lexsort((pos, rows))]
    gnp, gt = _np_grad(rng.standard_normal((911, 24)).astype(np.float32), "f16")
    _check(G, gnp, gt, rows, pos, 0, m, R, "f16", atomic_too=False)
    check_atomic(G, gnp, gt, rows, pos, R, "f16")


@pytest.mark.parametrize("dt,D", [("bf16", 72), ("f32", 132)])
def test_update_leaves_the_walk_only_repeated_rows(G, dt, D):
    """The backward with the optimizer step over more than 1024 chunks, against the two calls it stands for."""
    import paper_2301_02959_amd as fs
    rng = np.random.default_rng(D)
    R, n, m = 400_000, 2_000, 1024 * CHUNK + 300
    rows, _ = lookups(rng, m, R)
    pos = (np.arange(m) // (m // n + 1)).astype(np.int32)
    tdt = {"bf16": torch.bfloat16, "f32": torch.float32}[dt]
    grad = torch.randn(n, D, generator=torch.Generator().manual_seed(1)).to(tdt).to(G.DEV)
    table = torch.randn(R, D, generator=torch.Generator().manual_seed(2)).to(tdt).to(G.DEV)
    srows, spos = (torch.zeros(m, dtype=torch.int32, device=G.DEV) for _ in range(2))
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    fs.fs_sort_lookups(G.to_dev(rows, torch.int64), G.to_dev(pos), 0, m, R, n, srows, spos, st)
    got = []
    for fused in (True, False):
        w, state = table.clone(), torch.zeros(R, device=G.DEV)
        uniq = torch.zeros(m, dtype=torch.int64, device=G.DEV)
        rg = torch.zeros(m, D, device=G.DEV)
        nu = torch.zeros(1, dtype=torch.int64, device=G.DEV)
        if fused:
            fs.fs_seq_grad_bwd_update(grad, srows, spos, m, R, w, fs.FS_OPT_ADAGRAD_ROWWISE, 0.05, 1e-6, state, None, None, 0,
                                      uniq, rg, m, nu, st)
        else:
            fs.fs_seq_grad_bwd_sorted(grad, srows, spos, m, R, 0, uniq, rg, m, nu, st)
            fs.fs_sparse_update(w, uniq, rg, m, nu, fs.FS_OPT_ADAGRAD_ROWWISE, 0.05, 1e-6, state, dev_status=st)
        torch.cuda.synchronize()
        got.append((w, state, uniq[:int(nu.item())]))
    assert int(st.item()) == 0 and len(got[0][2]) == len(np.unique(rows))
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("D", [4, 64, 72, 128, 132, 256, 260])
@pytest.mark.parametrize("first", [0, 100])
def test_runs_over_many_chunks(G, D, first):
    """Runs that go on into 1, 2, 8, 9, 31 .. 130 further chunks: every length at which the fold's rounds change, for
    rows of one, two and four columns to a lane."""
    rng = np.random.default_rng(D + first)
    more = [1, 2, 7, 8, 9, 10, 16, 17, 31, 32, 33, 40, 63, 64, 65, 96, 127, 128, 129, 130, 300]
    rows = np.repeat(np.arange(len(more) + 1), [first] + [k * CHUNK for k in more])
    rows = rows[rows > 0] if first == 0 else rows
    m = len(rows)
    pos = (np.arange(m) % 1021).astype(np.int32)
    pos = pos[np.lexsort((pos, rows))]
    gnp, gt = _np_grad(rng.standard_normal((1021, D)).astype(np.float32), "f32")
    _check(G, gnp, gt, rows, pos, 0, m, len(more) + 2, "f32", atomic_too=False)


@pytest.mark.parametrize("D", [36, 60, 128, 132, 260])
@pytest.mark.parametrize("first", [0, 100])
def test_runs_left_to_the_long_fold(G, D, first):
    """Batches of more than a million chunks times columns: runs of up to 64 further chunks are folded by their own wave, longer
    ones by a block 256 carries at a time, 32 of them at once, for 32 columns each."""
    rng = np.random.default_rng(D + first)
    more = [1, 63, 64, 65, 66, 96, 97, 98, 255, 256, 257, 289, 512, 513, 514, 769, 1025]
    more.append(max(600, 1_000_000 // D + 2 - sum(more)))
    rows = np.repeat(np.arange(len(more) + 1), [first] + [k * CHUNK for k in more])
    rows = rows[rows > 0] if first == 0 else rows
    m = len(rows)
    assert -(-m // CHUNK) * D > 1_000_000
    pos = (np.arange(m) % 1021).astype(np.int32)
    pos = pos[np.lexsort((pos, rows))]
    gnp, gt = _np_grad(rng.standard_normal((1021, D)).astype(np.float32), "f32")
    _check(G, gnp, gt, rows, pos, 0, m, len(more) + 2, "f32", atomic_too=False)


@pytest.mark.parametrize("D,chunks", [(8, 9), (128, 70), (128, 7900), (256, 4100)])
@pytest.mark.parametrize("order", ["alternating", "long and short", "random"])
def test_rows_that_come_again(G, D, chunks, order):
    """Lists that are not ascending: every stretch of equal rows is a row of its own, wherever else its row stands, also
    where runs go on over many chunks; the workspace is not written past its end.  Gradients are small whole numbers."""
    import ctypes
    import paper_2301_02959_amd as fs
    m = chunks * CHUNK - 3
    k = torch.arange(m, device=G.DEV)
    if order == "alternating":                             # every chunk starts with row 7, every other one is nothing else
        rows = torch.where(k % (2 * CHUNK) <= CHUNK, 7, 9)
    elif order == "long and short":                        # 65 chunks of row 7 and a bit, then 65 that only start with it
        rows = torch.where((k % (130 * CHUNK) <= 65 * CHUNK) | (k % CHUNK == 0), 7, 9)
    else:
        gen = torch.Generator(device=G.DEV).manual_seed(chunks)
        rows = torch.randint(0, 3, (m // 200 + 1,), device=G.DEV, generator=gen).repeat_interleave(200)[:m]
    heads = torch.ones(m, dtype=torch.bool, device=G.DEV)
    heads[1:] = rows[1:] != rows[:-1]
    run = torch.cumsum(heads, 0) - 1
    runs = int(run[-1]) + 1
    pos = torch.arange(m, dtype=torch.int32, device=G.DEV) % 977
    grad = torch.randint(-2, 3, (977, D), device=G.DEV).float()
    want = torch.zeros(runs, D, device=G.DEV, dtype=torch.float64)
    for k0 in range(0, m, 1 << 20):
        want.index_add_(0, run[k0:k0 + (1 << 20)], grad[pos[k0:k0 + (1 << 20)].long()].double())
    uniq = torch.full((runs,), -7, dtype=torch.int64, device=G.DEV)
    rg = torch.full((runs, D), 7.0, device=G.DEV)
    nu = torch.zeros(1, dtype=torch.int64, device=G.DEV)
    st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    args = (m, 100, 0, uniq, rg, runs, nu, st)
    need = ctypes.c_size_t(0)
    assert fs._typed().fs_seq_grad_bwd_sorted(None, 977, D, fs.FS_F32, None, None, m, 100, 0, None, None, runs, None, None,
                                              ctypes.byref(need), None, None) == 0
    guarded = torch.full((need.value + (1 << 20),), 85, dtype=torch.uint8, device=G.DEV)
    fs.fs_seq_grad_bwd_sorted(grad, rows.to(torch.int32), pos, *args, workspace=guarded[:need.value])
    assert int(nu.item()) == runs
    assert bool(int(st.item()) & fs.FS_DEV_NOT_SORTED) == bool((rows[1:] < rows[:-1]).any())
    assert torch.equal(uniq, rows[heads]) and torch.equal(rg.double(), want)
    assert bool((guarded[need.value:] == 85).all())


@pytest.mark.parametrize("blocks", [1, 2, 3, 31, 32, 33])
@pytest.mark.parametrize("more", [-1, 0, 1])
@pytest.mark.parametrize("R", [50, 400_000])
def test_counting_blocks(G, blocks, more, R):
    """Up to 32 blocks of 64 chunks every wave adds up the blocks' run counts itself, beyond them a launch scans them; the
    number of runs with room for all of them and for fewer."""
    import paper_2301_02959_amd as fs
    m = blocks * 64 * CHUNK + more
    rows = torch.sort(torch.randint(0, R, (m,), device=G.DEV, generator=torch.Generator(device=G.DEV).manual_seed(m)))[0]
    pos = torch.arange(m, dtype=torch.int32, device=G.DEV) % 977                # ascending within a row is not needed for whole numbers
    grad = torch.randint(-2, 3, (977, 8), device=G.DEV).float()
    want_rows, inverse = torch.unique(rows, return_inverse=True)
    want = torch.zeros(len(want_rows), 8, device=G.DEV, dtype=torch.float64).index_add_(0, inverse, grad[pos.long()].double())
    for cap in (len(want_rows), len(want_rows) // 2):
        uniq = torch.full((cap + 1,), -7, dtype=torch.int64, device=G.DEV)
        rg = torch.full((cap + 1, 8), 7.0, device=G.DEV)
        nu = torch.zeros(1, dtype=torch.int64, device=G.DEV)
        st = torch.zeros(1, dtype=torch.int32, device=G.DEV)
        fs.fs_seq_grad_bwd_sorted(grad, rows.to(torch.int32), pos, m, R, 0, uniq, rg, cap, nu, st)
        assert int(nu.item()) == len(want_rows)
        assert bool(int(st.item()) & fs.FS_DEV_UNIQUE_OVERFLOW) == (cap < len(want_rows))
        assert torch.equal(uniq[:cap], want_rows[:cap]) and int(uniq[cap]) == -7
        assert torch.equal(rg[:cap].double(), want[:cap]) and bool((rg[cap] == 7.0).all())


@pytest.mark.parametrize("tail", [1, 2, 700])
@pytest.mark.parametrize("m", [1, 2, 300, 700, 1024 * CHUNK, 1024 * CHUNK + 1, 1024 * CHUNK + 300])
def test_last_row_of_all_ones(G, m, tail):
    """A caller's sorted list that ends with rows of 0xFFFFFFFF (-1, a padding value): outside the table, reported, and a
    row like any other for the sums.  The oracle sums it under the first number past the table."""
    import paper_2301_02959_amd as fs
    tail = min(tail, m)
    rng = np.random.default_rng(m + tail)
    R, n, D = 100_000, 1_500, 24
    rows = np.sort(np.concatenate([rng.integers(0, R, m - tail), np.full(tail, R)]))
    pos = (np.arange(m) // (m // n + 1)).astype(np.int32)
    gnp, gt = _np_grad(rng.standard_normal((n, D)).astype(np.float32), "f16")
    orc, ost, ou, og, _, onu = oracle.seq_grad_bwd(gnp, rows, pos, 0, m, R + 1, dtype=G.oracle_dtype("f16"))
    assert (orc, ost) == (0, 0)
    ou = np.where(ou == R, 0xFFFFFFFF, ou)
    srows = G.to_dev(np.where(rows == R, -1, rows), torch.int32)
    spos, grad = G.to_dev(pos), gt.to(G.DEV)

    def outputs():
        return (torch.full((onu,), 5, dtype=torch.int64, device=G.DEV), torch.full((onu, D), 7.0, device=G.DEV),
                torch.zeros(1, dtype=torch.int64, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV))

    uniq, rg, nu, st = outputs()
    fs.fs_seq_grad_bwd_sorted(grad, srows, spos, m, R, 0, uniq, rg, onu, nu, st)
    assert int(nu.item()) == onu and int(st.item()) == oracle.BAD_ID
    assert np.array_equal(uniq.cpu().numpy(), ou) and np.array_equal(G.bits(rg), og.view(np.uint8).reshape(-1))
    # the backward with the optimizer step skips that row and leaves every other one as the two calls do
    table = torch.randn(R, D, generator=torch.Generator().manual_seed(m)).to(torch.float16).to(G.DEV)
    two, w, state = table.clone(), table.clone(), [torch.zeros(R, device=G.DEV) for _ in range(2)]
    fs.fs_sparse_update(two, uniq, rg, onu, nu, fs.FS_OPT_ADAGRAD_ROWWISE, 0.05, 1e-6, state[0])
    uniq, rg, nu, st = outputs()
    scratch = torch.zeros(64 << 20, dtype=torch.uint8, device=G.DEV)
    fs.fs_seq_grad_bwd_update(grad, srows, spos, m, R, w, fs.FS_OPT_ADAGRAD_ROWWISE, 0.05, 1e-6, state[1], None, None, 0,
                              uniq, rg, onu, nu, st, workspace=scratch)
    assert int(nu.item()) == onu and int(st.item()) & oracle.BAD_ID
    assert np.array_equal(uniq.cpu().numpy(), ou)
    assert torch.equal(w.view(torch.int16), two.view(torch.int16)) and torch.equal(state[0], state[1])
