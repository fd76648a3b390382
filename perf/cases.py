"""The work that users of the tiered sequence-embedding lookup have it do, as measurable cases.

Every case is one program that calls the package's public entry points in the order in which a training or
serving loop calls them.  Which calls those are is the case's "path":

  serve      inference: route a jagged batch, gather its rows.
  exchange   the same on one GPU of several: the router hands over the replica slots, the GPU's own bucket is
             gathered from table and replica store, the rows of the other buckets go through the two halves of
             the row exchange (send buffer on the owner's side, placement on the requester's).
  step       one step of the benchmark: histogram of the batch and choice of the rows to replicate, route, sort,
             gather, backward over the shared sort.
  train      a training iteration with the optimizer applied by the backward pass: route, gather, sort, backward
             with update (table, optimizer state and replica store in place).
  forward    forward of a large batch in row order: route, sort, gather over the sorted pairs.
  backward   backward of a routed batch, sorting for itself.
  profile    the planning pass: histogram of a profiling sample from zero, then the rows that fit the budget.
  replan     new placement from a profile: tier cuts, replica store and its slots written into the placement.

Shapes are those of the repository's five configurations (or a stated share of them), ids are Zipf-like over a
random permutation of the rows, tables and gradients normal.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2301_02959_amd as fs

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ELEM = {"f32": 4, "f16": 2, "bf16": 2}
UNIT = {"f32": 4, "f16": 8, "bf16": 8}          # elements in 16 bytes: D is a multiple of this
OPTIMIZERS = {"sgd": fs.FS_OPT_SGD, "adagrad": fs.FS_OPT_ADAGRAD, "rowwise": fs.FS_OPT_ADAGRAD_ROWWISE}
TIER_GROUP, TIER_SHARDED = 1, 2


def _case(path, T, E, D, dtype, B, law, alpha, U, W, f0, f1=0.0, **more):
    """T tables of E rows x D; B samples with lengths of `law` ("name:arguments"); Zipf exponent alpha; U buckets
    in groups of W; f0 / f1: share of each table's rows (by popularity) that is replicated / kept per group."""
    return dict(path=path, T=T, E=E, D=D, dtype=dtype, B=B, law=law, alpha=alpha, U=U, W=W, f0=f0, f1=f1, **more)


def listed():
    cases = {
        # the smallest configuration, served: latency and launches are all there is
        "serve_smallest": _case("serve", 1, 100_000, 64, "f32", 256, "fixed:32", 1.05, 8, 8, 0.01),
        # an odd-sized serving request on one GPU of 64 in 8 groups, three tiers
        "exchange_ragged": _case("exchange", 4, 1_000_003, 128, "bf16", 173, "geometric:120:1024", 1.2, 64, 8, 0.002, 0.02),
        # the smallest configuration, one whole benchmark step
        "step_smallest": _case("step", 1, 100_000, 64, "f32", 256, "fixed:32", 1.05, 8, 8, 0.01, order="bucket"),
        # a small training batch with rows of an odd number of 16-byte pieces, element-wise optimizer
        "train_small_odd": _case("train", 3, 250_000, 72, "f16", 517, "uniform:1:64", 1.1, 24, 8, 0.005, 0.02, opt="adagrad"),
        # about a million lookups, row-wise optimizer, replica store mirrored
        "train_mid": _case("train", 8, 500_000, 128, "bf16", 1024, "uniform:1:256", 1.1, 64, 64, 0.005, opt="rowwise"),
        # second configuration: 8 tables of 10 M fp16 rows of 256 bytes, 4.2 M lookups; row order is the faster one
        "step_c2": _case("step", 8, 10_000_000, 128, "f16", 4096, "uniform:1:256", 1.1, 64, 64, 0.005, order="row"),
        # third configuration, the headline: 16 tables of 5 M bf16 rows of 512 bytes, 15.7 M lookups, three tiers
        "step_c3": _case("step", 16, 5_000_000, 256, "bf16", 8192, "geometric:120:1024", 1.2, 64, 8, 0.002, 0.02, order="bucket"),
        # the largest configuration's forward, a quarter of its batch over a quarter of its rows (18 M lookups)
        "forward_large": _case("forward", 16, 5_000_000, 256, "f16", 4096, "lognormal:5.3:0.8:2048", 1.1, 128, 128, 0.01),
        # its backward in full: 72 M lookups over 320 M rows
        "backward_largest": _case("backward", 16, 20_000_000, 256, "f16", 16384, "lognormal:5.3:0.8:2048", 1.1, 128, 128, 0.01),
        # fifth configuration's batch: extreme skew, a table's head row gathers a quarter of its lookups
        "backward_skewed": _case("backward", 4, 50_000_000, 128, "f16", 8192, "uniform:1:512", 1.3, 64, 64, 0.001),
        # its planning pass: 10^9 sampled ids over 4 x 50 M rows, top-k under 4 GB of 256-byte rows
        "profile_1e9": _case("profile", 4, 50_000_000, 128, "f16", 1, "around:250000000", 1.3, 64, 64, 0.001, budget=4_000_000_000),
        # new tiers for 8 tables of the third configuration from a profile of 32 M ids, store of 1 % of the rows
        "replan_tiers": _case("replan", 8, 5_000_000, 256, "bf16", 1, "around:4000000", 1.2, 64, 8, 0.002, 0.02, store=0.01),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, ragged, odd row widths among them."""
    path = rng.choice(["serve", "exchange", "step", "step", "train", "train", "forward", "backward", "backward", "profile", "replan"])

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    dtype = rng.choice(["f32", "f16", "bf16"])
    pieces = rng.choice([3, 4, 8, 9, 13, 16, 16, 24, 32, 32, 64])      # 48 to 1024 bytes per row
    D = pieces * UNIT[dtype]
    T = rng.choice([1, 2, 3, 4, 8, 16])
    E = log(20_000, 5_000_000)
    while T * E * D * ELEM[dtype] > 12e9:
        E //= 2
    U, W = rng.choice([(8, 8), (24, 8), (64, 8), (64, 64), (128, 128)])
    alpha = rng.choice([1.05, 1.1, 1.2, 1.3])
    mean = rng.choice([20, 60, 120, 250])
    law = rng.choice(["uniform:1:%d" % (2 * mean), "geometric:%d:%d" % (mean, 8 * mean), "lognormal:%g:0.8:2048" % (math.log(mean) - 0.32)])
    lookups = log(5_000, 10_000_000)
    while lookups * D * ELEM[dtype] > 6e9:
        lookups //= 2
    B = max(1, lookups // (T * mean))
    more = {}
    if path == "step":
        more["order"] = rng.choice(["bucket", "row"])
    if path == "train":
        more["opt"] = rng.choice(["sgd", "adagrad", "rowwise"])
    if path == "profile":
        B, law = 1, "around:%d" % (log(1_000_000, 300_000_000) // T)
        more["budget"] = log(20_000, 2_000_000) * D * ELEM[dtype]
    if path == "replan":
        B, law = 1, "around:%d" % (log(1_000_000, 50_000_000) // T)
        more["store"] = rng.choice([0.002, 0.01])
    return _case(path, T, E, D, dtype, B, law, alpha, U, W, rng.choice([0.002, 0.005, 0.01]), 0.02 if W < U else 0.0, **more)


# ---- inputs --------------------------------------------------------------------------------------------------

def _mean_length(law):
    name, *a = law.split(":")
    a = [float(x) for x in a]
    if name in ("fixed", "around"):
        return a[0]
    if name == "uniform":
        return (a[0] + a[1]) / 2
    if name == "geometric":
        return a[0] * (1 - math.exp(-a[1] / a[0]))
    return math.exp(a[0] + a[1] * a[1] / 2)


def _lengths(law, count, gen):
    name, *a = law.split(":")
    a = [float(x) for x in a]
    if name == "fixed":
        return torch.full((count,), int(a[0]), dtype=torch.int64, device=DEV)
    u = torch.rand(count, generator=gen, device=DEV, dtype=torch.float64)
    if name == "around":
        return (a[0] * (0.98 + 0.02 * u)).to(torch.int64)
    if name == "uniform":
        return (a[0] + torch.floor(u * (a[1] - a[0] + 1))).to(torch.int64)
    if name == "geometric":
        return (1 + torch.floor(torch.log1p(-u) / math.log(1 - 1 / a[0]))).clamp(1, a[1]).to(torch.int64)
    z = torch.randn(count, generator=gen, device=DEV, dtype=torch.float64)
    return torch.round(torch.exp(a[0] + a[1] * z)).clamp(1, a[2]).to(torch.int64)


def _ranks(count, E, alpha, gen):
    """Popularity ranks 0 .. E-1, P(rank r) the integral of x^-alpha over [r + 1/2, r + 3/2): a Zipf law within a
    few per cent at the head and exact in the tail, drawn without a table (so the same on every run)."""
    b = 1.0 - alpha
    lo, hi = 0.5 ** b, (E + 0.5) ** b
    u = torch.rand(count, generator=gen, device=DEV, dtype=torch.float64)
    x = u.mul_(hi - lo).add_(lo).pow_(1.0 / b)
    return x.sub_(0.5).floor_().clamp_(0, E - 1).to(torch.int64)


def _normal(shape, dtype, std, gen):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    step = 1 << 28
    for lo in range(0, flat.numel(), step):
        part = flat[lo:lo + step]
        part.copy_(torch.randn(part.numel(), generator=gen, device=DEV, dtype=torch.float32) * std)
    return out


def _batch(c, gen, with_placement=True):
    T, B, E = c["T"], c["B"], c["E"]
    # one multiset of lengths per shape, dealt to the segments by the seed: every batch of a case has the same size
    fixed = torch.Generator(device=DEV)
    fixed.manual_seed(2959 + T * B)
    lengths = _lengths(c["law"], T * B, fixed)[torch.randperm(T * B, generator=gen, device=DEV)]
    offsets = torch.zeros(T * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lengths, 0, out=offsets[1:])
    bounds = offsets[::B].tolist()
    n = bounds[-1]
    ids = torch.empty(n, dtype=torch.int64, device=DEV)
    placement = torch.empty(T * E, dtype=torch.int32, device=DEV) if with_placement else None
    if with_placement:
        local = torch.arange(E, dtype=torch.int64, device=DEV)
        sharded = ((TIER_SHARDED << 30) | (local % c["U"])).to(torch.int32)
    n0, n1 = int(c["f0"] * E), int(c["f1"] * E)
    for t in range(T):
        perm = torch.randperm(E, generator=gen, device=DEV)
        step = 1 << 27
        for lo in range(bounds[t], bounds[t + 1], step):
            hi = min(lo + step, bounds[t + 1])
            ids[lo:hi] = perm[_ranks(hi - lo, E, c["alpha"], gen)]
        if with_placement:
            entry = placement[t * E:(t + 1) * E]
            entry.copy_(sharded)
            entry[perm[n0:n0 + n1]] = ((TIER_GROUP << 30) | (perm[n0:n0 + n1] % c["W"])).to(torch.int32)
            entry[perm[:n0]] = 0
    row_base = torch.arange(T + 1, dtype=torch.int64, device=DEV) * E
    return dict(ids=ids, offsets=offsets, row_base=row_base, placement=placement, n=n)


def _zeros(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _distinct(c):
    """Expected number of distinct rows of the batch: per table the sum over ranks of 1 - (1 - p)^lookups."""
    E, a = c["E"], c["alpha"]
    m = c["B"] * _mean_length(c["law"])
    b = 1.0 - a
    norm = 0.5 ** b - (E + 0.5) ** b
    edge = np.unique(np.round(np.concatenate([np.arange(0, min(E, 2000) + 1), np.geomspace(1, E, 6000)])))
    mass = ((edge[:-1] + 0.5) ** b - (edge[1:] + 0.5) ** b) / norm
    width = np.diff(edge)
    return float(c["T"] * np.sum(width * -np.expm1(m * np.log1p(-np.minimum(mass / width, 1 - 1e-12)))))


def _capacity(c, n):
    return int(min(n, 1.15 * _distinct(c) + 4096))


def _workspace(query):
    """A workspace of the size that the C entry point asks for (its size query: workspace NULL)."""
    size = ctypes.c_size_t(0)
    assert query(ctypes.byref(size)) == 0
    return torch.empty(max(int(size.value), 256), dtype=torch.uint8, device=DEV)


def _route_workspace(c, n):
    return torch.empty(max(fs.route_workspace_bytes(c["T"], c["B"], n, c["U"], c["W"], 0), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 2959)
    T, E, D, B, U, W = (c[k] for k in ("T", "E", "D", "B", "U", "W"))
    R, dt, path = T * E, DTYPES[c["dtype"]], c["path"]
    s = dict(c=c, R=R, status=_zeros(1, torch.int32))
    s.update(_batch(c, gen, with_placement=path != "profile"))
    n = s["n"]
    if path == "profile":
        s.update(counts=_zeros(R, torch.int32), sel=_zeros(min(R, c["budget"] // (D * ELEM[c["dtype"]])), torch.int64), num_selected=_zeros(1, torch.int64))
        return s
    if path in ("serve", "exchange", "step", "train", "forward", "replan"):
        s["weights"] = _normal((R, D), dt, 0.1, gen)
    if path == "replan":
        s.update(counts=_zeros(R, torch.int32), cuts=_zeros(fs.FS_TIER_CUTS, torch.int64), slot_of_row=_zeros(R, torch.int32))
        s["k"] = int(c["store"] * R)
        s.update(rows=_zeros(s["k"], torch.int64), store=_zeros((s["k"], D), dt))
        fs.fs_plan_replication(s["ids"], s["offsets"], T, B, s["row_base"], n, R, s["counts"], fs.FS_PLAN_ACCUMULATE)
        # B samples of mean length 120 per GPU; the profile's ids are num_samples samples of that length per table
        s["params"] = dict(num_samples=max(1, n // T // 120), B=8192, U=U, W=W, dp_multiplier=6, granule=32,
                           a2a_global=1, a2a_intra=6, ar_global=3, ar_cross=2)
        return s
    s.update(bucket_offsets=_zeros(U + 1, torch.int64), rows=_zeros(n, torch.int64), pos=_zeros(n, torch.int32), tiers=_zeros(3, torch.int64))
    if path in ("exchange", "train"):
        # the replica store of the rows that the placement replicates, slots written into the placement
        chosen = torch.nonzero((s["placement"] >> 30) == 0).view(-1)
        s["k"] = int(chosen.numel())
        s.update(store=_zeros((s["k"], D), dt), slot_of_row=_zeros(R, torch.int32))
        fs.fs_replica_build(s["weights"], chosen, s["k"], None, s["store"], s["slot_of_row"])
        fs.fs_replica_tag_slots(s["placement"], s["slot_of_row"])
    if path != "backward":
        s["out"] = _zeros((n, D), dt)
    if path in ("serve", "forward"):
        s["ws_route"] = _route_workspace(c, n)
    if path == "exchange":
        s["slots"] = _zeros(n, torch.int32)
        fs.fs_route_bucketize_slots(s["ids"], s["offsets"], T, B, s["row_base"], s["placement"], n, U, W, 0,
                                    s["bucket_offsets"], s["rows"], s["pos"], s["slots"])
        s["own"] = int(s["bucket_offsets"][1])             # the ranks have exchanged their counts: known on the host
        s["send"] = _zeros((n, D), dt)                     # room for any split of the batch
    if path in ("step", "train", "backward"):
        s["grad"] = _normal((n, D), dt, 1.0, gen)
        cap = _capacity(c, n)
        s.update(cap=cap, uniq=_zeros(cap, torch.int64), row_grads=_zeros((cap, D), torch.float32), num_unique=_zeros(1, torch.int64))
    if path in ("step", "train", "forward"):
        s.update(srows=_zeros(n, torch.int32), spos=_zeros(n, torch.int32))
    if path == "step":
        s["budget_rows"] = max(1, int(c["f0"] * R))
        s.update(counts=_zeros(R, torch.int32), sel=_zeros(s["budget_rows"], torch.int64), num_selected=_zeros(1, torch.int64))
    if path == "train":
        s["state"] = _zeros({"sgd": 1, "rowwise": R, "adagrad": (R, D)}[c["opt"]], torch.float32)
    if path == "backward":
        fs.fs_route_bucketize(s["ids"], s["offsets"], T, B, s["row_base"], s["placement"], n, U, W, 0, s["bucket_offsets"], s["rows"], s["pos"])
        s["ids"] = s["placement"] = None                   # the forward pass is over
    return s


# ---- one pass ------------------------------------------------------------------------------------------------

def _route(s, workspace=None):
    c = s["c"]
    fs.fs_route_bucketize(s["ids"], s["offsets"], c["T"], c["B"], s["row_base"], s["placement"], s["n"], c["U"], c["W"], 0,
                          s["bucket_offsets"], s["rows"], s["pos"], s["tiers"], s["status"], workspace=workspace)


def _answer(s, *names):
    return {k: s[k] for k in names + ("status",)}


ROUTED = ("bucket_offsets", "rows", "pos", "tiers")


def run(s):
    c, n, R, st = s["c"], s["n"], s["R"], s["status"]
    path = c["path"]
    if path == "serve":
        _route(s, s["ws_route"])
        fs.fs_seq_gather_fwd(s["weights"], s["rows"], s["pos"], 0, n, s["out"], st)
        return _answer(s, "out", *ROUTED)
    if path == "exchange":
        fs.fs_route_bucketize_slots(s["ids"], s["offsets"], c["T"], c["B"], s["row_base"], s["placement"], n, c["U"], c["W"], 0,
                                    s["bucket_offsets"], s["rows"], s["pos"], s["slots"], s["tiers"], st)
        fs.fs_seq_gather_send(s["weights"], s["rows"], s["own"], n, s["send"], st)
        fs.fs_seq_gather_fwd_slots(s["weights"], s["store"], s["k"], s["rows"], s["slots"], s["pos"], 0, s["own"], s["out"], st)
        fs.fs_seq_unbucketize(s["send"], s["pos"], s["own"], n, s["out"], st)
        return _answer(s, "out", "send", "slots", *ROUTED)
    if path == "step":
        row_bytes = c["D"] * ELEM[c["dtype"]]
        fs.fs_plan_replication(s["ids"], s["offsets"], c["T"], c["B"], s["row_base"], n, R, s["counts"],
                               fs.FS_PLAN_ACCUMULATE | fs.FS_PLAN_SELECT, s["budget_rows"] * row_bytes, row_bytes,
                               s["sel"], s["num_selected"], None, st)
        _route(s)
        fs.fs_sort_lookups(s["rows"], s["pos"], 0, n, R, n, s["srows"], s["spos"], st)
        if c["order"] == "bucket":
            fs.fs_seq_gather_fwd(s["weights"], s["rows"], s["pos"], 0, n, s["out"], st)
        else:
            fs.fs_seq_gather_fwd_sorted(s["weights"], s["srows"], s["spos"], n, s["out"], st)
        fs.fs_seq_grad_bwd_sorted(s["grad"], s["srows"], s["spos"], n, R, 0, s["uniq"], s["row_grads"], s["cap"], s["num_unique"], st)
        return _answer(s, "out", "counts", "sel", "num_selected", "srows", "spos", "uniq", "row_grads", "num_unique", *ROUTED)
    if path == "train":
        _route(s)
        fs.fs_seq_gather_fwd(s["weights"], s["rows"], s["pos"], 0, n, s["out"], st)
        fs.fs_sort_lookups(s["rows"], s["pos"], 0, n, R, n, s["srows"], s["spos"], st)
        fs.fs_seq_grad_bwd_update(s["grad"], s["srows"], s["spos"], n, R, s["weights"], OPTIMIZERS[c["opt"]], 0.01, 1e-8,
                                  None if c["opt"] == "sgd" else s["state"], s["store"], s["slot_of_row"], s["k"],
                                  s["uniq"], s["row_grads"], s["cap"], s["num_unique"], st)
        return _answer(s, "out", "weights", "state", "store", "uniq", "num_unique", *ROUTED)
    if path == "forward":
        _route(s, s["ws_route"])
        fs.fs_sort_lookups(s["rows"], s["pos"], 0, n, R, n, s["srows"], s["spos"], st)
        fs.fs_seq_gather_fwd_sorted(s["weights"], s["srows"], s["spos"], n, s["out"], st)
        return _answer(s, "out", "srows", "spos", *ROUTED)
    if path == "backward":
        fs.fs_seq_grad_bwd(s["grad"], s["rows"], s["pos"], 0, n, R, 0, s["uniq"], s["row_grads"], s["cap"], s["num_unique"], st)
        return _answer(s, "uniq", "row_grads", "num_unique")
    if path == "profile":
        row_bytes = c["D"] * ELEM[c["dtype"]]
        s["counts"].zero_()
        fs.fs_plan_replication(s["ids"], s["offsets"], c["T"], c["B"], s["row_base"], n, R, s["counts"], fs.FS_PLAN_ACCUMULATE, dev_status=st)
        fs.fs_plan_replication(s["ids"], s["offsets"], c["T"], c["B"], s["row_base"], n, R, s["counts"], fs.FS_PLAN_SELECT,
                               c["budget"], row_bytes, s["sel"], s["num_selected"], None, st)
        return _answer(s, "counts", "sel", "num_selected")
    fs.fs_plan_tiers(s["counts"], R, s["params"], 3, s["rows"], s["k"], s["cuts"], s["placement"], st)
    fs.fs_replica_build(s["weights"], s["rows"], s["k"], s["cuts"][fs.FS_CUT_N_DP:fs.FS_CUT_N_DP + 1], s["store"], s["slot_of_row"], st)
    fs.fs_replica_tag_slots(s["placement"], s["slot_of_row"], st)
    return _answer(s, "rows", "cuts", "placement", "store", "slot_of_row")


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def work(case):
    """Bytes: each input read once and each output written once, rows that repeat in a batch fetched once.  Flops:
    the adds of the backward and the update's arithmetic (nothing here is a contraction)."""
    c = dict(case)
    n = c["T"] * c["B"] * _mean_length(c["law"])
    R, row = c["T"] * c["E"], c["D"] * ELEM[c["dtype"]]
    d = _distinct(c)
    path = c["path"]
    route = n * (8 + 8 + 4) + d * 4                          # id in, row and position out, a placement entry per distinct row
    forward = d * row + n * row                              # each distinct row in, every lookup's row out
    pairs = n * 8                                            # sorted pairs written
    back = n * row + d * (c["D"] * 4 + 8)                    # every lookup's gradient row in, a row sum and its index out
    plan = R * 4 + n * 8 + d * 8                             # counters read once, ids in, touched counters in and out
    adds = n * c["D"]
    if path == "serve":
        return {"bytes": route + forward, "flops": 0}
    if path == "exchange":
        return {"bytes": route + n * 4 + forward, "flops": 0}
    if path == "step":
        return {"bytes": plan + route + pairs + forward + back, "flops": adds}
    if path == "train":
        state = {"sgd": 0, "rowwise": 8, "adagrad": 8 * c["D"]}[c["opt"]]
        return {"bytes": route + pairs + forward + n * row + d * (2 * row + state + 8), "flops": adds + 6 * d * c["D"]}
    if path == "forward":
        return {"bytes": route + pairs + forward, "flops": 0}
    if path == "backward":
        return {"bytes": n * 12 + back, "flops": adds}
    if path == "profile":
        k = min(d, c["budget"] // row)
        return {"bytes": R * 8 + n * 8 + d * 8 + k * 8, "flops": 0}
    k = c["store"] * R
    return {"bytes": R * 4 + R * 4 + R * 8 + min(d, k) * (8 + 2 * row), "flops": 0}   # counters in, slots out, placement in and out, the store


def tolerance(case):
    """Everything but the optimizer step is defined to the bit: copies, indices, counts, and row gradients whose
    order of summation the interface states.  The update is fp32 arithmetic rounded once to the table's type."""
    if case["path"] != "train":
        return "exact"
    # against the same rules in 64 bits, sums in another order: weights and state 4e-7 (fp32), 5e-6 (16-bit table)
    return {"rel": 2e-6 if case["dtype"] == "f32" else 2e-5, "differ": 0.0}
