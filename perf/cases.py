"""The work a user of this framework has it do, as cases that can be timed and compared.

A case is one pass through the public entry points:

  step     one training iteration of a ranking model, all shards in one batched worker step
           (set_batch, worker_step_all, aggregate, apply_update)
  workers  the same iteration with one worker_step call per worker, the slowest workers left out of
           the aggregation when `left_out` > 0
  push     one worker's step on its shard and the gradients it pushes (the batch time of one worker)
  adam     the dense data-parallel step: weighted average of the workers' gradients and Adam

Batches, dense features, labels, MLP weights and optimizer state come from the seed; the embedding
tables get the framework's procedural initial values.  Optimizer state is that of a run under way
(accumulators of the size of a squared gradient), not the zeros of its first step.
"""
import math
from functools import lru_cache
from types import SimpleNamespace

import numpy as np
import torch

import paper_2404_09679_amd as A

DEV = "cuda"


# ---------------------------------------------------------------------------- the cases
def _model(kind, fields, rows, dim, batch, shards, hidden, *, table="f32", state="elementwise", num_dense=13,
           gemm="bf16", bag_min=1, bag_max=20, zipf=1.1, pooling="sum", split="equal", left_out=0, worker=0,
           own_streams=True):
    return dict(kind=kind, fields=fields, rows=rows, dim=dim, batch=batch, shards=shards, hidden=hidden, table=table,
                state=state, num_dense=num_dense, gemm=gemm, bag_min=bag_min, bag_max=bag_max, zipf=zipf,
                pooling=pooling, split=split, left_out=left_out, worker=worker, own_streams=own_streams)


def _adam(n, shards):
    return dict(kind="adam", n=n, shards=shards)


BIG_MLP, LARGE_MLP, TINY_MLP, MID_MLP = "1024-512-256", "1024-512", "64-32", "256-128"


def listed():
    return [
        # the smallest model, fp32 throughout: launches and their gaps are the whole cost
        dict(name="tiny-fp32", **_model("step", 8, 10_000, 16, 256, 4, TINY_MLP, gemm="f32", bag_max=4, zipf=1.05)),
        # a click-log ranking model on a small global batch of three workers (frequent synchronisation)
        dict(name="ranking-small-batch", **_model("step", 26, 1_000_000, 32, 96, 3, BIG_MLP)),
        # the same model at its ordinary global batch, eight equal workers
        dict(name="ranking", **_model("step", 26, 1_000_000, 32, 4096, 8, BIG_MLP)),
        # workers of different speed: a large odd batch split in proportion to the speeds
        dict(name="ranking-hetero", **_model("step", 26, 1_000_000, 32, 15_625, 8, BIG_MLP, split="speeds")),
        # workers stepping one by one, the servers disregarding the slowest one
        dict(name="ranking-backup", **_model("workers", 26, 1_000_000, 32, 3000, 6, BIG_MLP, left_out=1)),
        # mean-pooled bags (some of them empty), fp32 products, every kernel on the caller's stream
        dict(name="mean-fp32", **_model("step", 12, 100_000, 32, 1500, 5, MID_MLP, gemm="f32", bag_min=0, bag_max=12,
                                        pooling="mean", split="speeds", own_streams=False)),
        # large tables in bf16 with one accumulator per row, long bags, sixteen workers
        dict(name="large-bf16", **_model("step", 100, 1_200_000, 64, 16_384, 16, LARGE_MLP, table="bf16",
                                         state="rowwise", num_dense=0, bag_max=50, zipf=1.2)),
        # fewer fields and a ragged batch of the same kind of model
        dict(name="bf16-ragged", **_model("step", 60, 500_000, 64, 2501, 16, LARGE_MLP, table="bf16", state="rowwise",
                                          num_dense=0, bag_max=50, zipf=1.2, split="speeds")),
        # one worker's push on a small and on an ordinary shard
        dict(name="push-small", **_model("push", 26, 1_000_000, 32, 4096, 2, BIG_MLP, worker=64)),
        dict(name="push", **_model("push", 26, 1_000_000, 32, 4096, 2, BIG_MLP, worker=1531)),
        # dense step: a small model of odd size, and the largest one
        dict(name="adam-small", **_adam(1_000_003, 4)),
        dict(name="adam-large", **_adam(1 << 28, 8)),
    ]


def draw(rng):
    """One more case: the family of a listed case with its sizes and options drawn over their range."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    family = rng.choice(["tiny", "ranking", "ranking", "fp32", "bf16", "push", "adam"])
    split = rng.choice(["equal", "speeds"])
    if family == "tiny":
        return _model("step", rng.randint(4, 16), log_int(1000, 50_000), rng.choice([16, 32]), log_int(16, 1024),
                      rng.randint(1, 8), TINY_MLP, gemm="f32", bag_max=rng.randint(2, 8), zipf=1.05, split=split,
                      pooling=rng.choice(["sum", "mean"]))
    if family == "ranking":
        kind = rng.choice(["step", "step", "workers"])
        shards = rng.randint(3, 12)
        return _model(kind, rng.randint(10, 39), log_int(100_000, 1_000_000), rng.choice([16, 32, 64]),
                      log_int(64, 12_000 if kind == "step" else 6000), shards, BIG_MLP, bag_max=rng.randint(5, 20),
                      split=split, left_out=rng.randint(0, 2) if kind == "workers" else 0)
    if family == "fp32":
        return _model("step", rng.randint(6, 20), log_int(10_000, 200_000), rng.choice([16, 32]), log_int(128, 4096),
                      rng.randint(1, 10), MID_MLP, gemm="f32", bag_min=rng.choice([0, 1]), bag_max=rng.randint(4, 16),
                      pooling=rng.choice(["sum", "mean"]), split=split, own_streams=rng.choice([True, False]))
    if family == "bf16":
        return _model("step", rng.randint(30, 100), log_int(200_000, 1_200_000), 64, log_int(1000, 12_000),
                      rng.randint(4, 24), LARGE_MLP, table="bf16", state="rowwise", num_dense=0,
                      bag_max=rng.randint(20, 50), zipf=1.2, split=split)
    if family == "push":
        return _model("push", rng.randint(10, 39), log_int(100_000, 1_000_000), rng.choice([16, 32]), 4096, 2, BIG_MLP,
                      bag_max=rng.randint(5, 20), worker=log_int(8, 3072))
    return _adam(log_int(100_000, 100_000_000), rng.randint(1, 16))


# ---------------------------------------------------------------------------- inputs
@lru_cache(maxsize=4)
def _zipf_cdf(rows, s):
    """Bounded Zipf(s) over the ranks 1 .. rows (what the ids of a click log look like)."""
    c = np.cumsum(np.arange(1, rows + 1, dtype=np.float64) ** -s)
    return torch.from_numpy(c / c[-1]).to(DEV)


def _widths(case):
    hidden = [int(w) for w in case["hidden"].split("-")]
    return [case["fields"] * case["dim"] + case["num_dense"]] + hidden + [1]


def _speeds(n):
    """Measured speeds of n workers, the fastest eight times the slowest."""
    return [1.0 + 7.0 * k / max(1, n - 1) for k in range(n)]


def _included(case):
    """Which workers the servers aggregate: the first `left_out` (the slowest) are disregarded."""
    return [0 if k < case["left_out"] else 1 for k in range(case["shards"])]


def _batch(case, g):
    F, R, B = case["fields"], case["rows"], case["batch"]
    lens = torch.randint(case["bag_min"], case["bag_max"] + 1, (F, B), generator=g, device=DEV)
    offsets = torch.zeros((F, B + 1), dtype=torch.int32, device=DEV)
    offsets[:, 1:] = torch.cumsum(lens, 1)
    field_ptr = [0] + torch.cumsum(offsets[:, -1].long(), 0).tolist()
    cdf = _zipf_cdf(R, case["zipf"])
    ids = torch.empty(field_ptr[-1], dtype=torch.int32, device=DEV)
    for f in range(F):
        u = torch.rand(field_ptr[f + 1] - field_ptr[f], generator=g, device=DEV, dtype=torch.float64)
        rank = torch.searchsorted(cdf, u).clamp_(max=R - 1)
        mul = (2654435761 * (f + 1)) % R | 1   # a bijection rank -> row: hot rows are scattered as hashing does
        while math.gcd(mul, R) != 1:
            mul += 2
        ids[field_ptr[f]:field_ptr[f + 1]] = ((rank * mul + 7919 * f) % R).int()
    dense = torch.randn((B, case["num_dense"]), generator=g, device=DEV) if case["num_dense"] else None
    labels = (torch.rand(B, generator=g, device=DEV) < 0.25).float()
    return ids, field_ptr, offsets, dense, labels


def _mlp(widths, g):
    parts = []
    for i, o in zip(widths[:-1], widths[1:]):
        parts.append(torch.randn(i * o, generator=g, device=DEV) * math.sqrt(2.0 / i))
        parts.append(torch.randn(o, generator=g, device=DEV) * 0.01)
    return torch.cat(parts)


def _prepare_model(case, g):
    F, R, D, B, K = case["fields"], case["rows"], case["dim"], case["batch"], case["shards"]
    cfg = SimpleNamespace(num_fields=F, rows_per_field=R, dim=D, table_dtype=case["table"], adagrad_state=case["state"],
                          num_dense=case["num_dense"], layer_sizes=_widths(case), gemm_dtype=case["gemm"], lr=0.01,
                          eps=1e-8, shard_sizes=[0] * K, max_bag=case["bag_max"], pooling=case["pooling"])
    batch = _batch(case, g)
    tables = torch.empty((F * R, D), dtype=torch.bfloat16 if case["table"] == "bf16" else torch.float32, device=DEV)
    A.fill_tables(tables, F, R, D, 0.05)
    tstate = torch.rand((F * R,) if case["state"] == "rowwise" else (F * R, D), generator=g, device=DEV)
    tstate.add_(0.5).mul_((0.3 / B) ** 2)
    params = _mlp(cfg.layer_sizes, g)
    pstate = (torch.rand(params.shape, generator=g, device=DEV) + 0.5) * (0.02 ** 2 / B)
    mean_bag = 0.5 * (case["bag_min"] + case["bag_max"])   # the capacity covers any batch of these bags
    spread = case["bag_max"] / math.sqrt(12.0)
    capacity = int(F * B * mean_bag + 8 * spread * math.sqrt(F * B)) + 64
    ctx = A.Context(A.model_from_config(cfg, max_batch=B, max_nnz=max(capacity, batch[1][-1]), max_shards=K))
    if case["kind"] == "push":
        ctx.set_eager_weight_gradients(True)   # a worker's batch time includes its weight gradients
    if not case["own_streams"]:
        ctx.set_library_streams(False)
    ctx.bind(tables, tstate, params, pstate)
    if case["kind"] == "push":
        ctx.assign_shard(B, 2, sizes=[B - case["worker"], case["worker"]])
    elif case["split"] == "speeds":
        ctx.assign_shard(B, K, speed=_speeds(K))
    else:
        ctx.assign_shard(B, K)
    loss = torch.zeros(K, device=DEV)
    return SimpleNamespace(case=case, ctx=ctx, batch=batch, tables=tables, tstate=tstate, params=params, pstate=pstate,
                           loss=loss, losses=[loss[k:k + 1] for k in range(K)], mask=_included(case))


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if case["kind"] != "adam":
        return _prepare_model(case, g)
    n, K = case["n"], case["shards"]
    p = torch.randn(n, generator=g, device=DEV) * 0.02
    m = torch.randn(n, generator=g, device=DEV) * 1e-3
    v = torch.rand(n, generator=g, device=DEV) * 2e-6
    grads = [torch.randn(n, generator=g, device=DEV) * 1e-3 for _ in range(K)]
    speeds = _speeds(K)
    weights = [s / sum(speeds) for s in speeds]
    return SimpleNamespace(case=case, p=p, m=m, v=v, grads=grads, weights=weights)


# ---------------------------------------------------------------------------- one pass
def run(state):
    kind = state.case["kind"]
    if kind == "adam":
        A.dense_aggregate_adam(state.p, state.m, state.v, state.grads, state.weights, 1e-3, 0.9, 0.999, 1e-8, 100)
        return {"p": state.p, "m": state.m, "v": state.v}
    ctx = state.ctx
    ctx.set_batch(*state.batch)
    if kind == "push":
        ctx.worker_step(1, state.losses[1])
        dense, dx = ctx.view_shard_grads(1)
        return {"loss": state.losses[1], "dense": dense, "dx": dx}
    if kind == "step":
        ctx.worker_step_all(state.loss)
        ctx.aggregate()
    else:
        for k, on in enumerate(state.mask):
            if on:
                ctx.worker_step(k, state.losses[k])
        ctx.aggregate(state.mask if state.case["left_out"] else None)
    ctx.apply_update()
    return {"loss": state.loss, "params": state.params, "pstate": state.pstate, "tables": state.tables,
            "tstate": state.tstate}


# ---------------------------------------------------------------------------- what a pass cannot do without
def _samples(case):
    """Samples a pass works on (expected, where a split decides)."""
    B, K = case["batch"], case["shards"]
    if case["kind"] == "push":
        return case["worker"]
    if case["split"] == "speeds":
        s = _speeds(K)
        return int(B * sum(v for v, on in zip(s, _included(case)) if on) / sum(s))
    return B * sum(_included(case)) // K


@lru_cache(maxsize=64)
def _distinct_rows(rows, s, lookups):
    """Expected number of distinct rows among `lookups` draws of the bounded Zipf."""
    p = np.arange(1, rows + 1, dtype=np.float64) ** -s
    return float(-np.expm1(lookups * np.log1p(-p / p.sum())).sum())


def work(case):
    if case["kind"] == "adam":
        n, K = case["n"], case["shards"]
        return {"bytes": 4.0 * n * (K + 3 + 3), "flops": n * (2.0 * K + 16)}
    F, D, n = case["fields"], case["dim"], _samples(case)
    lookups = n * 0.5 * (case["bag_min"] + case["bag_max"])           # per field
    distinct = F * _distinct_rows(case["rows"], case["zipf"], lookups)
    row = D * (2 if case["table"] == "bf16" else 4)
    state = 4 if case["state"] == "rowwise" else 4 * D
    w = _widths(case)
    P = sum(i * o + o for i, o in zip(w[:-1], w[1:]))
    weights = sum(i * o for i, o in zip(w[:-1], w[1:]))
    batch = 4.0 * F * lookups + 4.0 * F * n + 4.0 * n * (case["num_dense"] + 1)
    flops = 6.0 * n * weights + 3.0 * F * lookups * D
    if case["kind"] == "push":   # rows and parameters read, dense and pooled-input gradients written
        return {"bytes": batch + distinct * row + 8.0 * P + 4.0 * n * F * D, "flops": flops - 2.0 * F * lookups * D}
    return {"bytes": batch + 2.0 * distinct * (row + state) + 16.0 * P, "flops": flops}


def tolerance(case):
    """About four times the largest error measured on the outputs against the same pass in 64 bits
    (with bf16 products: with every stored bf16 value rounded there too).  What is left with bf16 are
    values that round to another bf16 neighbour when a sum is formed in another order, and now and
    then a unit whose ReLU decision changes with it: single entries, hence the wider `max`."""
    if case["kind"] == "adam":
        return {"rel": 5e-7, "max": 2e-6}
    if case["gemm"] == "f32":
        return {"rel": 2e-6, "max": 1e-5}
    if case["kind"] == "push":     # the gradients themselves, not steps on parameters
        return {"rel": 1.3e-2, "max": 0.95}
    return {"rel": 2e-3, "max": 0.2}
