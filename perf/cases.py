"""The calls whose time counts, as a program that uses the layer makes them.

A case is one of five kinds of work:

  lookup    the forward alone (serving, evaluation): ``pool_fwd``
  step      a training step: ``Layer.step`` (forward, dedup, reduce + update)
  backward  the dedup, the gradient rows and a separate optimizer step
            (programs that inspect, clip or exchange gradient rows before the
            update): ``unique_ids``, ``grad_reduce``, ``sparse_update``
  pipeline  consecutive training steps on the pipelined schedule:
            ``Pipeline.run``
  route     the send order of a batch over the ranks of a sharded layer:
            ``route_ids``

Shapes are those of the synthetic workloads this repository benchmarks and
tests (one small table; 8 tables of 1M rows; one table of 50M rows; 26 tables
of mixed sizes in bf16; long-tailed ids), with tables of at most 13 GB so that
an updated table can be returned whole.
"""
import math

import numpy as np
import torch

import paper_2112_02752_amd as emb

_DEV = "cuda"

# Fields of a case (defaults; a case states what differs):
#   tables      number of stacked tables
#   rows_lo/hi  rows of the smallest and largest table, spaced evenly in their logarithm
#   dim, dtype  row width and table type ("fp32" or "bf16")
#   bags        bags per table
#   lens        bag lengths: "uniform" 1..lmax, "poisson" (mean lam, clamped to 1..lmax), "onehot",
#               "mixed" (even tables one-hot, odd ones uniform 1..lmax)
#   empty       share of bags left empty
#   zipf        exponent of the ids' bounded Zipf law (0: uniform); tables under 200k rows of a
#               many-table case take uniform ids
#   id_bits     32 or 64
#   pool, opt, rounding, concurrent: the layer's options
#   steps       training steps of one pipelined call
#   ranks       ranks of a sharding
_DEFAULTS = dict(tables=1, rows_lo=0, rows_hi=0, dim=64, dtype="fp32", bags=0, lens="uniform", lmax=20, lam=0.0,
                 empty=0.0, zipf=1.05, id_bits=32, pool="sum", opt="sgd", rounding="nearest", concurrent="no", steps=1,
                 ranks=1)

_LR, _EPS, _H0_EW = 0.01, 1e-8, 0.1


def _case(name, kind, **kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    c["kind"] = kind
    if name:
        c["name"] = name
    return c


def listed():
    one_50m = dict(rows_lo=50_000_000, rows_hi=50_000_000, dim=64, bags=16384, lens="poisson", lam=30.0, lmax=200,
                   zipf=1.2, opt="adagrad")
    mixed_26 = dict(tables=26, rows_lo=1000, rows_hi=10_000_000, dim=128, dtype="bf16", bags=8192, lens="mixed",
                    lmax=100, zipf=1.05, opt="adagrad")
    small = dict(rows_lo=100_000, rows_hi=100_000, dim=16, bags=512, lmax=20, zipf=1.05)
    return [
        # serving: a request of a few hundred bags, where the call's latency is all there is
        _case("lookup_small", "lookup", **small),
        # serving or evaluation of a many-table model, bf16 tables
        _case("lookup_26tables_bf16", "lookup", **mixed_26),
        # a small training step (a CTR batch of 512): bound by latency and launches
        _case("step_small", "step", **small),
        # one-hot categorical features, wide rows, a batch that is no power of two
        _case("step_onehot_wide", "step", tables=3, rows_lo=20_000, rows_hi=2_000_000, dim=256, bags=6007,
              lens="onehot", zipf=1.05, opt="adagrad"),
        # an ordinary step over several tables with mean pooling
        _case("step_8tables_mean", "step", tables=8, rows_lo=1_000_000, rows_hi=1_000_000, dim=64, bags=4096, lmax=50,
              zipf=1.1, pool="mean", opt="adagrad"),
        # the benchmarked table, one step after another
        _case("step_50m", "step", **one_50m),
        # the benchmarked table on the pipelined schedule
        _case("pipeline_50m", "pipeline", steps=24, **one_50m),
        # bf16 training with the options that keep it accurate: element-wise Adagrad, stochastic rounding;
        # int64 ids as PyTorch makes them, some bags empty, an odd row width and batch
        _case("step_bf16_elementwise", "step", tables=5, rows_lo=50_000, rows_hi=3_000_000, dim=104, dtype="bf16",
              bags=3001, lmax=40, empty=0.1, zipf=1.1, id_bits=64, pool="mean", opt="adagrad_ew",
              rounding="stochastic"),
        # the largest step: 26 tables, 5.5M lookups, bf16
        _case("step_26tables_bf16", "step", concurrent="auto", **mixed_26),
        # a long tail: most ids of a large batch are distinct
        _case("step_long_tail", "step", rows_lo=50_000_000, rows_hi=50_000_000, dim=64, bags=65536, lmax=100,
              zipf=0.9),
        # gradient rows made, then applied apart (int64 ids)
        _case("backward_8tables", "backward", tables=8, rows_lo=1_000_000, rows_hi=1_000_000, dim=64, bags=4096,
              lmax=50, zipf=1.1, id_bits=64, opt="adagrad"),
        # ids bucketed by owner before the exchange of a sharded layer
        _case("route_8ranks", "route", ranks=8, **one_50m),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lookup", "step", "step", "step", "backward", "pipeline", "route"])
    dtype = rng.choice(["fp32", "fp32", "bf16"])
    per16 = 4 if dtype == "fp32" else 8
    dim = per16 * max(1, _log_uniform(rng, 8, 512) // per16)
    tables = rng.choice([1, 1, 1, _log_uniform(rng, 2, 26)])
    lens = rng.choice(["uniform", "uniform", "poisson", "onehot", "mixed" if tables > 1 else "uniform"])
    lmax = _log_uniform(rng, 4, 100)
    mean_len = {"uniform": (lmax + 1) / 2, "poisson": 0.3 * lmax + 1, "onehot": 1.0,
                "mixed": (lmax + 3) / 4}[lens]
    steps = rng.randint(2, 20) if kind == "pipeline" else 1
    # lookups of a batch: from a few hundred to 2M, and no more than 96M gathered values a call
    n = _log_uniform(rng, 300, min(2_000_000, 96_000_000 // (dim * steps)))
    bags = max(1, int(n / (mean_len * tables)))
    # at most 4 GB of table
    most = 4_000_000_000 // (dim * 4 * tables)
    hi = _log_uniform(rng, min(2000, most), min(20_000_000, most))
    lo = hi if tables == 1 else _log_uniform(rng, max(10, hi // 1000), hi)
    return _case("", kind, tables=tables, rows_lo=lo, rows_hi=hi, dim=dim, dtype=dtype, bags=bags, lens=lens,
                 lmax=lmax, lam=0.3 * lmax + 1 if lens == "poisson" else 0.0, empty=rng.choice([0.0, 0.0, 0.2]),
                 zipf=rng.choice([0.0, 0.9, 1.05, 1.2]), id_bits=rng.choice([32, 32, 64]),
                 pool=rng.choice(["sum", "mean"]), opt=rng.choice(["sgd", "adagrad", "adagrad", "adagrad_ew"]),
                 rounding=rng.choice(["nearest", "stochastic"]) if dtype == "bf16" else "nearest",
                 concurrent=rng.choice(["no", "auto"]), steps=steps,
                 ranks=rng.choice([2, 8, 13, 64]) if kind == "route" else 1)


# ---------------------------------------------------------------- inputs

def _rows(case):
    T, lo, hi = case["tables"], case["rows_lo"], case["rows_hi"]
    if T == 1:
        return [hi]
    return [int(round(lo * (hi / lo) ** (t / (T - 1)))) for t in range(T)]


def _onehot(case, t):
    return case["lens"] == "onehot" or (case["lens"] == "mixed" and t % 2 == 0)


def _zipf_of(case, rows):
    return 0.0 if case["tables"] > 1 and rows < 200_000 else case["zipf"]


def _lengths(case, t, gen):
    B = case["bags"]
    if _onehot(case, t):
        n = torch.ones(B, dtype=torch.int64, device=_DEV)
    elif case["lens"] == "poisson":
        n = torch.poisson(torch.full((B,), case["lam"], device=_DEV), generator=gen).to(torch.int64)
        n = n.clamp(1, case["lmax"])
    else:
        n = torch.randint(1, case["lmax"] + 1, (B,), device=_DEV, generator=gen)
    if case["empty"] > 0:
        n[torch.rand(B, device=_DEV, generator=gen) < case["empty"]] = 0
    return n


def _ids(n, rows, s, gen):
    """n ids of a bounded Zipf(s) law over `rows` ranks (inverse of the law's continuous form), the ranks
    scattered over the rows by an affine bijection."""
    u = torch.rand(n, device=_DEV, generator=gen, dtype=torch.float64)
    if s == 0.0:
        return (u * rows).to(torch.int64).clamp_(0, rows - 1)
    a, b = 0.5 ** (1 - s), (rows + 0.5) ** (1 - s)
    rank = ((a + u * (b - a)) ** (1 / (1 - s)) - 0.5).to(torch.int64).clamp_(0, rows - 1)
    mul = 2_654_435_761 % rows or 1
    while math.gcd(mul, rows) != 1:
        mul += 1
    return (rank * mul + rows // 3) % rows


def _batch(case, gen):
    rows = _rows(case)
    lens = [_lengths(case, t, gen) for t in range(case["tables"])]
    off = torch.zeros(case["tables"] * case["bags"] + 1, dtype=torch.int64, device=_DEV)
    off[1:] = torch.cumsum(torch.cat(lens), 0)
    ids = [_ids(int(x.sum()), r, _zipf_of(case, r), gen) for x, r in zip(lens, rows)]
    idt = torch.int64 if case["id_bits"] == 64 else torch.int32
    return emb.Batch(off.to(torch.int32), torch.cat(ids).to(idt), case["bags"])


def _capacity(case):
    """Ids the buffers hold: a batch's expected number and ten standard deviations."""
    mean = var = 0.0
    for t in range(case["tables"]):
        if _onehot(case, t):
            m, v = 1.0, 0.0
        elif case["lens"] == "poisson":
            m, v = case["lam"] + 1.0, case["lam"] + 1.0
        else:
            m, v = (case["lmax"] + 1) / 2, (case["lmax"] ** 2 - 1) / 12
        mean += case["bags"] * m
        var += case["bags"] * (v + m * m * min(1.0, case["empty"]))
    return int(math.ceil(mean + 10 * math.sqrt(var)))


def _row_offset(case):
    return [0] + [int(x) for x in np.cumsum(_rows(case))]


def _inputs(case, seed):
    """Tables, optimizer state, and per step a batch with its upstream gradient."""
    gen = torch.Generator(device=_DEV)
    gen.manual_seed(seed)
    ro = _row_offset(case)
    R, D, M = ro[-1], case["dim"], case["tables"] * case["bags"]
    W = state = None
    if case["kind"] != "route":
        W = torch.empty((R, D), dtype=torch.float32 if case["dtype"] == "fp32" else torch.bfloat16, device=_DEV)
        W.uniform_(-0.01, 0.01, generator=gen)
        if case["kind"] != "lookup":
            if case["opt"] == "adagrad":
                state = torch.zeros(R, device=_DEV)
            elif case["opt"] == "adagrad_ew":
                state = torch.full((R, D), _H0_EW, device=_DEV)
    else:
        # the bucketing reads the tables' bounds, not their rows
        W = torch.zeros((1, D), device=_DEV)
    batches = [_batch(case, gen) for _ in range(case["steps"])]
    grads = [torch.randn((M, D), device=_DEV, generator=gen) for _ in batches] \
        if case["kind"] not in ("lookup", "route") else []
    return emb.Tables(W, ro), state, batches, grads


def _shard_start(case):
    R, n = _row_offset(case)[-1], case["ranks"]
    return [R * r // n for r in range(n + 1)]


def prepare(case, seed):
    tables, state, batches, grads = _inputs(case, seed)
    kind, D, M = case["kind"], case["dim"], case["tables"] * case["bags"]
    s = dict(case=case, tables=tables, state=state, batches=batches, grads=grads)
    n = _capacity(case)
    if kind in ("lookup", "step", "pipeline"):
        s["outs"] = [torch.zeros((M, D), device=_DEV) for _ in batches]
    opts = dict(pool=case["pool"], opt=case["opt"], lr=_LR, eps=_EPS, state=state, max_indices=n, max_bags=M,
                rounding=case["rounding"], seed=17)
    i32 = dict(dtype=torch.int32, device=_DEV)
    if kind == "step":
        s["layer"] = emb.Layer(tables, concurrent="auto" if case["concurrent"] == "auto" else False, **opts)
    elif kind == "pipeline":
        s["pipe"] = emb.Pipeline(tables, **opts)
    elif kind == "backward":
        s["dedup"] = emb.DedupBuffers(_DEV, n, M, D)
        s["grad_rows"] = torch.zeros((n, D), device=_DEV)
    elif kind == "route":
        s["shard_start"] = _shard_start(case)
        s["counts"] = torch.zeros(case["ranks"], **i32)
        s["send"] = [torch.zeros(n, **i32) for _ in range(3)]
        s["ws"] = torch.zeros(emb.route_workspace_size(n, M, case["ranks"]), dtype=torch.uint8, device=_DEV)
    return s


def run(s):
    case, tables, batch = s["case"], s["tables"], s["batches"][0]
    kind = case["kind"]
    if kind == "lookup":
        emb.pool_fwd(tables, batch, case["pool"], s["outs"][0])
        return {"out": s["outs"][0]}
    if kind == "step":
        s["layer"].step(batch, s["outs"][0], s["grads"][0])
        return {"out": s["outs"], "W": tables.weights, "state": s["state"]}
    if kind == "pipeline":
        s["pipe"].run(list(zip(s["batches"], s["outs"], s["grads"])))
        return {"out": s["outs"], "W": tables.weights, "state": s["state"]}
    if kind == "backward":
        d, rows = s["dedup"], s["grad_rows"]
        emb.unique_ids(tables, batch, d.unique_keys, d.counts, d.seg_offsets, d.sort_perm, d.num_unique, d.ws)
        emb.grad_reduce(tables, batch, case["pool"], s["grads"][0], d.sort_perm, d.seg_offsets, d.unique_keys,
                        d.num_unique, d.ws, grad_rows=rows)
        emb.sparse_update(tables, case["opt"], _LR, _EPS, s["state"], d.unique_keys, d.num_unique,
                          int(batch.indices.numel()), rows, rounding=case["rounding"], seed=17)
        return {"unique_keys": d.unique_keys, "counts": d.counts, "seg_offsets": d.seg_offsets,
                "sort_perm": d.sort_perm, "num_unique": d.num_unique, "grad_rows": rows, "W": tables.weights,
                "state": s["state"]}
    emb.route_ids(tables, batch, s["shard_start"], s["counts"], s["send"][0], s["send"][1], s["send"][2], s["ws"])
    return {"counts": s["counts"], "ids": s["send"][0], "pos": s["send"][1], "bag": s["send"][2]}


# ---------------------------------------------------------------- work

def _distinct(n, rows, s):
    """Expected number of distinct ids among n draws of _ids(n, rows, s)."""
    if n <= 0:
        return 0.0
    if s == 0.0:
        return rows * -math.expm1(n * math.log1p(-1.0 / rows)) if rows > 1 else 1.0
    edges = np.unique(np.concatenate([np.arange(0, min(rows, 1000) + 1),
                                      np.geomspace(min(rows, 1000), rows, 2000).round()])).astype(np.float64)
    x = (edges + 0.5) ** (1 - s)
    width = np.diff(edges)
    p = np.diff(x) / (x[-1] - x[0]) / width
    return float((width * -np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-12)))).sum())


def work(case):
    T, B, D = case["tables"], case["bags"], case["dim"]
    M = T * B
    N = U = 0.0
    for t, r in enumerate(_rows(case)):
        mean = 1.0 if _onehot(case, t) else case["lam"] if case["lens"] == "poisson" else (case["lmax"] + 1) / 2
        n = B * mean * (1 - case["empty"])
        N += n
        U += _distinct(n, r, _zipf_of(case, r))
    row = D * (4 if case["dtype"] == "fp32" else 2)
    st = {"sgd": 0, "adagrad": 4, "adagrad_ew": 4 * D}[case["opt"]]
    ids = 4.0 * (M + 1) + N * case["id_bits"] / 8
    kind = case["kind"]
    if kind == "route":
        return {"bytes": ids + 12 * N + 4 * case["ranks"], "flops": 0}
    if kind == "lookup":
        return {"bytes": ids + U * row + 4.0 * M * D, "flops": N * D}
    update = 2 * U * (row + st)                       # rows and state read and written
    if kind == "backward":
        outs = 4 * N + 12 * U + 4.0 * U * D           # permutation, runs, gradient rows
        return {"bytes": ids + 4.0 * M * D + update + outs, "flops": N * D + 6 * U * D}
    k = case["steps"]
    return {"bytes": k * (ids + 8.0 * M * D + update), "flops": k * (2 * N * D + 6 * U * D)}


def tolerance(case):
    if case["kind"] == "route":
        return "exact"
    if case["kind"] == "lookup":
        # fp32 sums of a bag's rows
        return {"rel": 4e-7, "max": 2e-5}
    # whole values (permutation, keys, counts) are the same; fp32 sums in another order
    if case["dtype"] == "fp32":
        return {"rel": 1e-6, "max": 1e-4, "differ": 0.0}
    # a stored bf16 value may fall on the other side of a rounding boundary (one unit in the last place)
    return {"rel": 1e-3, "max": 3e-2, "differ": 0.0}


# ---------------------------------------------------------------- 64 bits

def exact(case, seed):
    kind = case["kind"]
    if kind == "route":
        return None
    tables, state, batches, grads = _inputs(case, seed)
    ro, D, B = tables.row_offset, case["dim"], case["bags"]
    M = case["tables"] * B
    W = tables.weights.double()
    tables.weights = None
    H = state.double() if state is not None else None
    start = torch.tensor(ro[:-1], dtype=torch.int64, device=_DEV)
    outs, rows_out = [], None
    for k, b in enumerate(batches):
        off = b.offsets.to(torch.int64)
        n = off[1:] - off[:-1]
        bag = torch.repeat_interleave(torch.arange(M, device=_DEV), n)
        key = start[bag // B] + b.indices.to(torch.int64)
        scale = 1.0 / n.clamp(min=1).double() if case["pool"] == "mean" else torch.ones(M, device=_DEV).double()
        if kind != "backward":
            out = torch.zeros((M, D), dtype=torch.float64, device=_DEV)
            for c in torch.arange(len(key), device=_DEV).split(1 << 20):
                out.index_add_(0, bag[c], W[key[c]])
            outs.append(out * scale[:, None])
        if kind == "lookup":
            return {"out": outs[0]}
        keys, inv = torch.unique(key, return_inverse=True)
        g = torch.zeros((len(keys), D), dtype=torch.float64, device=_DEV)
        G = grads[k].double() * scale[:, None]
        for c in torch.arange(len(key), device=_DEV).split(1 << 20):
            g.index_add_(0, inv[c], G[bag[c]])
        if kind == "backward":
            rows_out = torch.zeros((_capacity(case), D), dtype=torch.float64, device=_DEV)
            rows_out[:len(keys)] = g
        if case["opt"] == "sgd":
            step = _LR * g
        elif case["opt"] == "adagrad":
            H[keys] += (g * g).mean(1)
            step = _LR * g / (H[keys].sqrt() + _EPS)[:, None]
        else:
            H[keys] += g * g
            step = _LR * g / (H[keys].sqrt() + _EPS)
        new = W[keys] - step
        # later steps of a call read the rows as the table's type holds them
        W[keys] = new if case["dtype"] == "fp32" or k == len(batches) - 1 else new.to(torch.bfloat16).double()
    if kind == "backward":
        return {"unique_keys": None, "counts": None, "seg_offsets": None, "sort_perm": None, "num_unique": None,
                "grad_rows": rows_out, "W": W, "state": H}
    return {"out": outs, "W": W, "state": H}
