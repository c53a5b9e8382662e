"""GPU parity of kernel variants at the sizes where their tiling can go wrong: one sample more or
fewer than a tile, remainders in every dimension, the smallest and largest problem a variant is
chosen for.  Same oracle and tolerances as test_gpu_parity.py."""
import dataclasses

import numpy as np
import pytest

import workload as wl
from test_gpu_parity import TOL32, TOLBF, check_iteration

pytestmark = pytest.mark.gpu


def _config(name, seed, **kw):
    base = dict(name=name, num_fields=3, rows_per_field=2000, dim=16, table_dtype="f32", adagrad_state="elementwise",
                num_dense=5, layer_sizes=None, gemm_dtype="bf16", max_bag=3, zipf_s=1.1, shard_sizes=(1,),
                seed=wl.SEED0 + seed)
    base.update(kw)
    width = base["num_fields"] * base["dim"] + base["num_dense"]
    base["layer_sizes"] = (width,) + tuple(base["layer_sizes"]) + (1,)
    return wl.RankingConfig(**base)


# (samples per shard, hidden widths): tiles of 32 (few blocks), 32 x 64, 64, 128 (two and three stages) and 256 rows and columns in
# the forward and data-gradient products, tiles of 64 and 128 in the weight gradients; no dimension a multiple of its tile
PRODUCT_SHAPES = [((1,), (8,)), ((20, 13), (40, 8)), ((151, 150), (1032, 264)), ((513, 0, 199), (264, 72)), ((1300, 801), (1544, 1160)),
                  ((2000, 1301), (1032, 136)), ((5003, 3200), (2056, 1544))]


@pytest.mark.parametrize("sizes,hidden", PRODUCT_SHAPES, ids=[str(sum(s)) for s, _ in PRODUCT_SHAPES])
def test_bf16_product_tiles(sizes, hidden):
    cfg = _config(f"tiles-{sum(sizes)}", 400 + sum(sizes), layer_sizes=hidden, shard_sizes=sizes)
    check_iteration(cfg, sizes, tol=TOLBF, bf16_gemm_oracle=True, batched=True, nonzero_state=True)


# the same for fp32 products: tiles of 16 and 32, widths that no vector load fits, fewer contraction slots than a step
F32_SHAPES = [((1,), (7,)), ((15, 17), (33, 5)), ((513, 0, 199), (64, 19)), ((2600, 1501), (520, 36))]


@pytest.mark.parametrize("sizes,hidden", F32_SHAPES, ids=[str(sum(s)) for s, _ in F32_SHAPES])
def test_f32_product_tiles(sizes, hidden):
    cfg = _config(f"f32-tiles-{sum(sizes)}", 500 + sum(sizes), layer_sizes=hidden, shard_sizes=sizes, gemm_dtype="f32")
    check_iteration(cfg, sizes, tol=TOL32, batched=True, nonzero_state=True)


def _plant(monkeypatch, field_ids, B, offsets_of):
    """Batches of every configuration carry these ids (one array per field) and offsets."""
    real = wl.make_batch
    offsets = np.stack([offsets_of(f, len(ids)) for f, ids in enumerate(field_ids)]).astype(np.int32)
    assert all(offsets[f, 0] == 0 and offsets[f, -1] == len(ids) and offsets.shape[1] == B + 1 for f, ids in enumerate(field_ids))
    ptr = np.cumsum([0] + [len(ids) for ids in field_ids]).astype(np.int64)
    ids = np.concatenate(field_ids).astype(np.int32)
    monkeypatch.setattr(wl, "make_batch", lambda c, index=0: dataclasses.replace(real(c, index), ids=ids, offsets=offsets, field_ptr=ptr))


# The reduction works on windows of 256 sorted lookups.  Runs in sorted order: long ones that end at, start at, fill
# and cross window boundaries, one that spans three windows; around 2048 a run of 16 (the longest that one lane group sums
# whole) and one of 17 (the shortest that is cut into pieces) over a boundary, runs of 1 .. 5, 15, 31 and 33; the field
# ends inside, one behind, at and one before the end of a window.
RUN_LENGTHS = [100, 156, 300, 212, 256, 513, 254, 1, 16, 17, 15, 31, 33, 1, 1, 2, 3, 4, 5, 28, 91, 16, 239, 17, 700, 1200]
ENDS = np.cumsum(RUN_LENGTHS)


@pytest.mark.parametrize("dim,table,state,more", [(4, "f32", "elementwise", 0), (32, "f32", "elementwise", 141), (256, "f32", "rowwise", 140),
                                                  (8, "bf16", "rowwise", 142), (64, "bf16", "elementwise", 255)])
def test_runs_and_windows(dim, table, state, more, monkeypatch):
    starts = ENDS - RUN_LENGTHS
    long = np.array(RUN_LENGTHS) > 16
    assert np.any(long & (ENDS % 256 == 0) & (starts % 256 != 0)) and np.any(long & (starts % 256 == 0) & (ENDS % 256 != 0))
    assert np.any((starts % 256 == 0) & (np.array(RUN_LENGTHS) == 256)) and np.any(ENDS // 256 - starts // 256 >= 3)
    assert any(n == 16 and e // 256 > st // 256 and e % 256 for n, st, e in zip(RUN_LENGTHS, starts, ENDS))
    assert any(n == 17 and e // 256 > st // 256 and e % 256 for n, st, e in zip(RUN_LENGTHS, starts, ENDS))
    assert [(int(ENDS[-1]) + m) % 256 for m in (140, 141, 142)] == [255, 0, 1]
    lengths = RUN_LENGTHS + [1] * more
    bag = 5
    total = sum(lengths)
    B = -(-total // bag)
    cfg = _config(f"windows-{dim}", 600 + dim, num_fields=2, rows_per_field=1200, dim=dim, table_dtype=table, adagrad_state=state,
                  layer_sizes=(8,), gemm_dtype="f32", shard_sizes=(B // 3, B - B // 3), max_bag=bag)
    rng = np.random.default_rng(7 + dim)
    ids = [rng.permutation(np.repeat(np.sort(rng.permutation(1200)[:len(lengths)]), lengths)) for _ in range(2)]
    _plant(monkeypatch, ids, B, lambda f, n: np.minimum(np.arange(B + 1) * bag, n))
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)


# The sort of a field in one block holds 2, 4, 8 or 16 lookups per thread, by the longest field; above, tiles of 2048 over
# many blocks.  One, two and three passes.
@pytest.mark.parametrize("most", [2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("rows", [1000, 70_000, 1_100_000])
def test_sort_variants(most, rows, monkeypatch):
    sizes = [most, most - 1, 0, 1, 1025, 1023]
    F, B = (6, 500) if rows < 1_000_000 else (2, 500)
    cfg = _config(f"sort-{most}", 610, num_fields=F, rows_per_field=rows, dim=4, layer_sizes=(8,), gemm_dtype="f32",
                  shard_sizes=(100, 0, 399, 1), max_bag=most // 400 + 1)
    rng = np.random.default_rng(most + rows)
    ids = [rng.integers(0, rows, n) // rng.integers(1, 9, n) for n in sizes[:F]]
    _plant(monkeypatch, ids, B, lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)


# bf16 models of a batched step: a pass of the sort in each of the first products' launches (tiles of 32 by four wavefronts, of 32 x 64 by eight and
# of 64), up to 4096 lookups of a field; one pass, two, and three where two launches are all there are (the aggregation then sorts).
@pytest.mark.parametrize("most", [1, 64, 257, 1025, 2048, 4096, 4097])
@pytest.mark.parametrize("rows,hidden", [(900, (40,)), (70_000, (520, 264)), (70_000, (1032, 8)), (1_100_000, (264,))])
def test_sort_beside_bf16_products(most, rows, hidden, monkeypatch):
    sizes = [most, most - 1, 0, 1, 255, 1023]
    F, B = (6, 500) if rows < 1_000_000 else (2, 500)
    cfg = _config(f"sort-bf16-{most}", 650, num_fields=F, rows_per_field=rows, dim=4, layer_sizes=hidden, shard_sizes=(100, 0, 399, 1),
                  max_bag=most // 400 + 1)
    rng = np.random.default_rng(most + rows)
    ids = [rng.integers(0, rows, n) // rng.integers(1, 9, n) for n in sizes[:F]]
    _plant(monkeypatch, ids, B, lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    check_iteration(cfg, cfg.shard_sizes, tol=TOLBF, bf16_gemm_oracle=True, batched=True, nonzero_state=True)


# Where a batched step of a bf16 model has its sort's passes beside the products: if as many of them have room for one.  Tiles of 128 have none, two
# products too few for three passes, and an input gradient in the launch of the weight gradients is no launch of its own; the aggregation then
# sorts, in one launch.
@pytest.mark.parametrize("fields,dim,samples,hidden,rows,eager,joins", [(26, 32, 96, (1024, 512, 256), 1_200_000, False, True), (24, 64, 4095, (1024,), 50_000, False, False),
                                                                       (24, 64, 4095, (1024, 64), 50_000, False, False), (24, 64, 4095, (1024, 64, 64), 50_000, False, True), (20, 64, 2000, (256,), 50_000, False, True),
                                                                       (20, 64, 2000, (256,), 1_200_000, False, False), (26, 32, 300, (256,), 50_000, True, False),
                                                                       (26, 32, 300, (256,), 900, True, True)])
def test_where_a_bf16_step_sorts(fields, dim, samples, hidden, rows, eager, joins):
    import torch
    import paper_2404_09679_amd as A
    dev = "cuda:0"
    cfg = _config(f"where-{samples}", 643, num_fields=fields, rows_per_field=rows, dim=dim, layer_sizes=hidden, num_dense=0, shard_sizes=(samples,), max_bag=1)
    g = torch.Generator(device=dev).manual_seed(samples)
    ids = torch.randint(0, rows, (fields, samples), generator=g, device=dev).int()
    tables = torch.zeros((fields * rows, dim), device=dev)
    params = torch.zeros(sum(i * o + o for i, o in zip(cfg.layer_sizes, cfg.layer_sizes[1:])), device=dev)
    ctx = A.Context(A.model_from_config(cfg, max_batch=samples, max_nnz=fields * samples, max_shards=1))
    ctx.set_eager_weight_gradients(eager)
    ctx.bind(tables, torch.ones_like(tables), params, torch.ones_like(params))
    ctx.set_batch(ids.flatten(), [f * samples for f in range(fields + 1)], torch.arange(samples + 1, dtype=torch.int32, device=dev).repeat(fields, 1), None,
                  torch.zeros(samples, device=dev))
    ctx.assign_shard(samples, 1)
    scatter = A.kernel_names().index("sort_scatter")
    ctx.worker_step_all(torch.zeros(1, device=dev))
    ctx.profile(2, scatter)
    ctx.aggregate()
    assert ctx.profile_read(scatter)[0] == (0 if joins else 1)
    ctx.profile(0)
    for f in range(fields):
        u, so, ss, _ = ctx.view_coalesced(f)
        key, order = torch.sort(ids[f], stable=True)
        rows_f, counts = torch.unique_consecutive(key, return_counts=True)
        assert torch.equal(u, rows_f) and torch.equal(so.long()[1:], torch.cumsum(counts, 0)) and torch.equal(ss.long(), order)


# The sort over many blocks (one field of more than 16384 lookups, ten tiles and a bit) with the other fields at the tile
# boundaries, before and after shards are left out, and anew after a new split; mean-pooled.  All of these sort in the
# aggregation; the long ones (of 100 000 lookups) of a batched step beside the MLP.
@pytest.mark.parametrize("how", ["batched", "by-worker", "masked", "masked-batched", "mean", "mean-masked", "new-split", "late-factors",
                                 "batched-long", "masked-batched-long", "mean-long", "new-split-long", "late-factors-long"])
def test_sort_over_many_blocks(how, monkeypatch):
    import torch
    sizes = [2048, 4096, 2049, 2047, 4095, 4097, 1, 0, 6144, 20_483, 2048]
    left = [2048, 2048, 1, 2047, 2048, 4097, 1, 0, 4096, 18_432, 0]      # ... of these in the first shard and the last
    long = how.endswith("-long")
    how = how[:-5] if long else how
    if long:
        sizes, left = sizes + [30_000, 30_721], left + [20_000, 28_673]
    assert (sum(sizes) >= 100_000) == long
    B, shards = 900, (300, 200, 400)
    cfg = _config(f"blocks-{how}", 620, num_fields=len(sizes), rows_per_field=5000, dim=8, layer_sizes=(8,), gemm_dtype="f32",
                  shard_sizes=shards, max_bag=24, pooling="mean" if how.startswith("mean") else "sum")
    rng = np.random.default_rng(13)

    def offsets(f, n):
        first = left[f] // 2
        cuts = [(0, first, 300), (first, first + n - left[f], 200), (first + n - left[f], n, 400)]
        parts = [np.concatenate([np.sort(rng.integers(lo, hi + 1, k - 1)), [hi]]) for lo, hi, k in cuts]
        return np.concatenate([[0]] + parts)

    ids = [rng.integers(0, 5000, n) // rng.integers(1, 60, n) for n in sizes]
    _plant(monkeypatch, ids, B, offsets)
    # (accumulators from zero: with others a step is about 1e-4 here, and rounding the stored parameter of about 0.05 to
    # fp32, 2^-25 * 0.05 = 1.5e-9, is 1.5e-5 of it: more than the 1e-5 that steps are compared to)
    kw = dict(tol=TOL32, batched=how not in ("by-worker", "masked", "mean-masked"))
    if "masked" in how:
        kw["mask"] = (1, 0, 1)
    if how == "late-factors":
        kw.update(scale=(0.5, 2.0, 1.0), scale_late=True)
    if how == "new-split":
        def prelude(run):
            run.ctx.assign_shard(B, 3)
            run.ctx.worker_step_all(torch.zeros(3, device="cuda:0"))
        kw.update(prelude=prelude, batched=False)
    check_iteration(cfg, shards, **kw)


# From three million lookups the sort does not wait for the gather, which then records no sample indices: what comes
# after must find them all the same.  From four million (rows of up to 32 columns) windows of 512 lookups.
@pytest.mark.parametrize("how,bag", [("masked", 20), ("late-factors", 20), ("mean", 27)])
def test_sort_ahead_of_the_gather(how, bag):
    B = 20_000
    cfg = _config(f"early-{how}", 630, num_fields=8, rows_per_field=3000, dim=4, layer_sizes=(8,), gemm_dtype="f32",
                  shard_sizes=(7000, 1, 4999, 8000), min_bag=bag - 1, max_bag=bag, pooling="mean" if how == "mean" else "sum")
    lookups = len(wl.make_batch(cfg).ids)
    assert lookups >= (3_000_000 if how != "mean" else 4 << 20)
    kw = {"masked": dict(mask=(1, 1, 0, 1)), "late-factors": dict(scale=(0.5, 2.0, 1.0, 1.5), scale_late=True), "mean": {}}[how]
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, **kw)   # (from zero accumulators: smaller steps than above)


# Large batches are sorted by buckets: rows cut where a sample of the lookups says.  From two million lookups of a batched step on if the passes
# are three (1.1 M rows) or the pooled inputs many (500 100 samples), else from 3.5 million, and of up to 2^18 rows from eight million; not
# where ranges that leave room for the sample in a word are too many (1.1 M rows, 500 100 samples).  Fields of many
# lookups, none, one and a few; ids spread evenly, by frequency, in the first rows, in one, in some that are neighbours, at both ends, past a
# multiple of 2^16 rows; buckets larger than a block holds (64 of them for 900 000 lookups of 1500 rows).  The sorted lookups are those
# of a stable sort, one for one.
# From eight million on the sort also works the samples out of the bags' boundaries: bags of one, empty ones, one of all.
KINDS = ["even", "zipf", "first-rows", "one-row", "neighbours", "ends", "past-65536"]


@pytest.mark.parametrize("rows", [1500, 70_001, 1_100_000])
@pytest.mark.parametrize("kind,B", [(k, 3001) for k in KINDS + ["even-8M", "zipf-8M"]] + [(k, 500_100) for k in KINDS + ["even-8M"]] +
                         [("even-8M", 65_536), ("even-8M", 65_537), ("ends-8M", 65_537), ("one-row-8M", 3001), ("first-rows-8M", 3001), ("past-65536-8M", 3001)])
def test_sort_by_buckets(kind, B, rows):
    import torch
    import paper_2404_09679_amd as A
    dev = "cuda:0"
    many = kind.endswith("-8M")
    kind, longest = (kind[:-3], 7_000_000) if many else (kind, 900_000)
    buckets = many or (B == 3001 and rows == 1_100_000) or B == 500_100
    if B == 500_100 and rows == 1_100_000:
        buckets = False
    sizes = [longest, 0, 700_001, 1, 8193, 500_000]
    cfg = _config(f"buckets-{kind}", 640, num_fields=len(sizes), rows_per_field=rows, dim=4, layer_sizes=(8,), gemm_dtype="f32", num_dense=0,
                  shard_sizes=(2000, B - 2000), max_bag=400)
    g = torch.Generator(device=dev).manual_seed(rows)
    draw = lambda lo, hi, n: torch.randint(lo, hi, (n,), generator=g, device=dev)

    def ids_of(n):
        if kind == "zipf":
            u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
            return ((u.clamp(min=1e-6) ** -1.5).long() * 7919) % rows
        if kind == "first-rows":
            return torch.minimum(draw(0, rows, n), draw(0, 40, n) ** 2 % rows)
        if kind == "one-row":
            return torch.full((n,), rows // 3, device=dev)
        if kind == "neighbours":
            return rows - 1 - draw(0, 12, n)
        if kind == "ends":
            return draw(0, 2, n) * (rows - 1)
        if kind == "past-65536":
            return (65_530 + draw(0, 13, n)) % rows
        return draw(0, rows, n)

    ids = [ids_of(n).int() for n in sizes]
    offsets = torch.zeros((len(sizes), B + 1), dtype=torch.int32, device=dev)
    for f, n in enumerate(sizes):
        cuts = draw(0, n + 1, B - 1)
        if f == 0:     # bags of one lookup, and empty ones
            cuts[:1000] = torch.arange(1000, device=dev) + 5000
            cuts[1000:1300] = 70_000
        if f == 5:     # one bag of nearly all
            cuts %= 100
        offsets[f, 1:B] = torch.sort(cuts)[0].int()
        offsets[f, B] = n
    tables = torch.randn((len(sizes) * rows, 4), generator=g, device=dev) * 0.05
    state = torch.ones_like(tables)
    params = torch.randn(sum(i * o + o for i, o in zip((24, 8), (8, 1))), generator=g, device=dev) * 0.3
    ctx = A.Context(A.model_from_config(cfg, max_batch=B, max_nnz=sum(sizes), max_shards=2))
    ctx.bind(tables, state, params, torch.ones_like(params))
    ptr = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    ctx.set_batch(torch.cat(ids), ptr, offsets, None, (torch.rand(B, generator=g, device=dev) < 0.25).float())
    ctx.assign_shard(B, 2, sizes=[2000, B - 2000])
    loss = torch.zeros(2, device=dev)
    sample = [torch.repeat_interleave(torch.arange(B, device=dev), (offsets[f, 1:] - offsets[f, :-1]).long()) for f in range(len(sizes))]

    def check(below):
        for f in range(len(sizes)):
            u, so, ss, _ = ctx.view_coalesced(f)
            on = sample[f] < below
            key, order = torch.sort(ids[f][on], stable=True)
            rows_f, counts = torch.unique_consecutive(key, return_counts=True)
            assert torch.equal(u.long(), rows_f.long()), (f, "rows")
            assert torch.equal(so.long()[1:], torch.cumsum(counts, 0)) and int(so[0]) == 0, (f, "runs")
            assert torch.equal(ss.long(), sample[f][on][order]), (f, "samples")

    scan = A.kernel_names().index("sort_scan")
    ctx.profile(2, scan)
    ctx.worker_step_all(loss)
    ctx.aggregate()
    assert ctx.profile_read(scan)[0] == (1 if buckets else 3 if rows == 1_100_000 else 2)
    ctx.profile(0)
    check(B)
    # what follows a batched step finds the samples it left out: a shard stepped anew, a shard left out
    ctx.worker_step_all(loss)
    ctx.worker_step(1, loss[1:])
    ctx.aggregate()
    check(B)
    ctx.worker_step_all(loss)
    ctx.aggregate([1, 0])
    check(2000)


# Bags of one length in a batch of a multiple of 1024 samples: evenly spaced lookups are then all at one place of their bags, and where the ids have
# an order in the bag, rows cut by those alone make ranges of most of the lookups, a block's work each.  The sort takes about as long
# as that of the same ids in random order (several times as long, were most in one range), and gives the same.
@pytest.mark.parametrize("B,bag,rows", [(16_384, 50, 50_000), (8192, 100, 1_100_000)])   # (more fields where fewer rows ask for more lookups)
@pytest.mark.parametrize("order", ["ascending", "first", "padded"])
def test_sort_by_buckets_of_bags_of_one_length(order, B, bag, rows):
    import torch
    import paper_2404_09679_amd as A
    dev, F = "cuda:0", 3 if rows > 1 << 20 else 10
    cfg = _config(f"bags-{bag}", 642, num_fields=F, rows_per_field=rows, dim=4, layer_sizes=(8,), gemm_dtype="f32", num_dense=0, shard_sizes=(B,), max_bag=bag)
    g = torch.Generator(device=dev).manual_seed(bag)
    even = torch.randint(0, rows, (F, B, bag), generator=g, device=dev).int()
    ids = {"ascending": torch.sort(even, dim=2)[0], "first": torch.cat([torch.full_like(even[:, :, :1], rows // 2), even[:, :, 1:]], 2),
           "padded": torch.where(torch.arange(bag, device=dev) < torch.randint(1, bag, (F, B, 1), generator=g, device=dev), even, 0)}[order]
    mixed = torch.stack([t.flatten()[torch.randperm(B * bag, generator=g, device=dev)] for t in ids]).flatten().contiguous()
    offsets = (torch.arange(B + 1, dtype=torch.int32, device=dev) * bag).repeat(F, 1).contiguous()
    tables = torch.randn((F * rows, 4), generator=g, device=dev) * 0.05
    params = torch.randn(sum(i * o + o for i, o in zip((4 * F, 8), (8, 1))), generator=g, device=dev) * 0.3
    ctx = A.Context(A.model_from_config(cfg, max_batch=B, max_nnz=F * B * bag, max_shards=1))
    ctx.bind(tables, torch.ones_like(tables), params, torch.ones_like(params))
    labels, loss = (torch.rand(B, generator=g, device=dev) < 0.25).float(), torch.zeros(1, device=dev)
    kid = A.kernel_names().index("sort_scatter")
    took = []
    for x in (mixed, ids.flatten().contiguous()):
        ctx.set_batch(x, [f * B * bag for f in range(F + 1)], offsets, None, labels)
        ctx.assign_shard(B, 1)
        times = []
        for _ in range(5):
            ctx.profile(2, kid)
            ctx.worker_step_all(loss)
            ctx.aggregate()
            times.append(ctx.profile_read(kid)[1])
            ctx.profile(0)
        took.append(min(times))
    for f in range(F):
        key, at = torch.sort(ids[f].flatten(), stable=True)
        u, so, ss, _ = ctx.view_coalesced(f)
        rows_f, counts = torch.unique_consecutive(key, return_counts=True)
        assert torch.equal(u, rows_f) and torch.equal(so.long()[1:], torch.cumsum(counts, 0)) and torch.equal(ss.long(), at // bag)
    assert took[1] < 2 * took[0], took


# An fp32 model without a hidden layer, whose loss kernel's sums share memory with what follows the worker step, and enough lookups that the sort
# beside it goes by buckets: sums that end where the reduction's memory has not ended, and (69 088 samples) where its last part, which the sort
# takes too, has begun.  Against float64.
@pytest.mark.parametrize("dim,B", [(16, 40_000), (4, 69_088)])
def test_sort_beside_a_model_without_hidden_layer(dim, B):
    import torch
    import paper_2404_09679_amd as A
    dev, F, rows, num_dense, sizes = "cuda:0", 2, 60_000, 4096, [900_001, 1_299_999]
    shards = [B // 2, 0, 7, B // 3, B - B // 2 - 7 - B // 3]
    cfg = _config(f"head-{B}", 641, num_fields=F, rows_per_field=rows, dim=dim, layer_sizes=(), gemm_dtype="f32", num_dense=num_dense,
                  shard_sizes=shards, max_bag=400)
    g = torch.Generator(device=dev).manual_seed(B)
    ids = [(torch.rand(n, generator=g, device=dev) ** 3 * rows).int() for n in sizes]
    offsets = torch.zeros((F, B + 1), dtype=torch.int32, device=dev)
    for f, n in enumerate(sizes):
        offsets[f, 1:B] = torch.sort(torch.randint(0, n + 1, (B - 1,), generator=g, device=dev))[0].int()
        offsets[f, B] = n
    width = F * dim + num_dense
    tables = torch.randn((F * rows, dim), generator=g, device=dev) * 0.05
    state = torch.full_like(tables, 1e-12)   # (accumulators as large as the squared gradients)
    params = torch.randn(width + 1, generator=g, device=dev) * width ** -0.5
    pstate = torch.full_like(params, 1e-5)
    dense = torch.randn((B, num_dense), generator=g, device=dev)
    labels = (torch.rand(B, generator=g, device=dev) < 0.25).float()
    ctx = A.Context(A.model_from_config(cfg, max_batch=B, max_nnz=sum(sizes), max_shards=len(shards)))
    ctx.bind(tables, state, params, pstate)
    ctx.set_batch(torch.cat(ids), [0, sizes[0], sum(sizes)], offsets, dense, labels)
    ctx.assign_shard(B, len(shards), sizes=shards)
    # the step in float64
    sample = [torch.repeat_interleave(torch.arange(B, device=dev), (offsets[f, 1:] - offsets[f, :-1]).long()) for f in range(F)]
    x = torch.zeros((B, width), dtype=torch.float64, device=dev)
    for f in range(F):
        x[:, f * dim:(f + 1) * dim].index_add_(0, sample[f], tables[f * rows + ids[f].long()].double())
    x[:, F * dim:] = dense
    w = params.double()
    z = x @ w[:width] + w[width]
    losses = torch.nn.functional.binary_cross_entropy_with_logits(z, labels.double(), reduction="none")
    starts = np.concatenate([[0], np.cumsum(shards)])
    dz = torch.sigmoid(z) - labels.double()
    want_loss, want_grad, total = [], torch.zeros(width + 1, dtype=torch.float64, device=dev), torch.zeros(B, dtype=torch.float64, device=dev)
    for k, n in enumerate(shards):
        at = slice(int(starts[k]), int(starts[k + 1]))
        want_loss.append(float(losses[at].mean()) if n else 0.0)
        want_grad += torch.cat([x[at].T @ dz[at], dz[at].sum()[None]]) / B   # (weight n / B, mean over n)
        total[at] = dz[at] / B
    rel = lambda a, b: float((a.double() - b).norm() / b.norm())
    old = tables.double()
    want = old.clone()
    for f in range(F):
        gr = torch.zeros((rows, dim), dtype=torch.float64, device=dev)
        gr.index_add_(0, ids[f].long(), total[sample[f]][:, None] * w[None, f * dim:(f + 1) * dim])
        want[f * rows:(f + 1) * rows] -= cfg.lr * gr / ((1e-12 + gr * gr).sqrt() + cfg.eps)
    loss = torch.zeros(len(shards), device=dev)
    for _ in range(3):
        ctx.worker_step_all(loss)
        ctx.aggregate()
        assert np.allclose(loss.cpu().numpy(), want_loss, rtol=1e-5)
        assert rel(ctx.view_dense_grad(), want_grad) < 1e-5
        for f in range(F):
            u, so, ss, _ = ctx.view_coalesced(f)
            key, order = torch.sort(ids[f], stable=True)
            rows_f, counts = torch.unique_consecutive(key, return_counts=True)
            assert torch.equal(u, rows_f) and torch.equal(so.long()[1:], torch.cumsum(counts, 0)) and torch.equal(ss.long(), sample[f][order])
    ctx.apply_update()
    torch.cuda.synchronize()
    # (a step grows no faster than its gradient; rows of 0.05 are rounded to 2e-9 behind steps of 1e-3 and more)
    assert rel(tables.double() - old, want - old) < 1e-5
    assert rel(w - params.double(), cfg.lr * want_grad / ((1e-5 + want_grad ** 2).sqrt() + cfg.eps)) < 1e-5


def test_gather_from_a_table_of_2_32_pieces():
    """2^30 rows of 64 bytes: places of rows no longer fit 32 bits.  Pooled inputs and updated rows against torch, the rows
    2^28, 2^29, ... away from the looked-up ones against their initial values."""
    import torch
    import paper_2404_09679_amd as A
    R, D, B, bag = 1 << 30, 16, 300, 4
    cfg = _config("wide-gather", 640, num_fields=1, rows_per_field=R, dim=D, num_dense=0, layer_sizes=(8,), gemm_dtype="f32",
                  adagrad_state="rowwise", shard_sizes=(B,), max_bag=bag)
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(3)
    tables = torch.empty((R, D), device=dev)
    A.fill_tables(tables, 1, R, D, 0.05)
    state = torch.ones(R, device=dev)
    params = torch.randn(D * 8 + 8 + 8 + 1, generator=g, device=dev) * 0.3
    ids = torch.randint(0, R, (B * bag,), generator=g, device=dev, dtype=torch.int32)
    ids[:4] = torch.tensor([R - 1, 0, R - 2, R // 2], dtype=torch.int32, device=dev)
    rows = ids.long()
    before = tables[rows]
    far = torch.cat([(rows + (1 << k)) % R for k in (26, 27, 28, 29)])
    far = far[~torch.isin(far, rows)]
    far_before = tables[far]
    ctx = A.Context(A.model_from_config(cfg, max_nnz=B * bag))
    ctx.bind(tables, state, params, torch.ones_like(params))
    offsets = torch.arange(0, B * bag + 1, bag, dtype=torch.int32, device=dev).reshape(1, -1)
    ctx.set_batch(ids, [0, B * bag], offsets, None, torch.ones(B, device=dev))
    ctx.assign_shard(B, 1)
    ctx.worker_step_all(torch.zeros(1, device=dev))
    ctx.aggregate()
    torch.cuda.synchronize()
    want = before.reshape(B, bag, D).sum(1)
    assert float((ctx.view_pooled(0) - want).abs().max()) <= 1e-6 * float(want.abs().max())
    unique, _, _, G = ctx.view_coalesced(0)
    assert torch.equal(unique.long(), torch.unique(rows))
    unique, G = unique.long().clone(), G.clone()
    old = tables[unique]
    ctx.apply_update()
    torch.cuda.synchronize()
    s1 = 1.0 + (G * G).mean(1, keepdim=True)
    want = old - cfg.lr * G / (s1.sqrt() + cfg.eps)
    assert float((tables[unique] - want).abs().max()) <= 1e-6 * float(old.abs().max()) and not torch.equal(tables[unique], old)
    assert torch.equal(tables[far], far_before) and bool((state[far] == 1).all())


# enough samples per shard that the weight gradients are formed piece by piece: unequal weights (a piece per shard, the
# longest first) and equal ones (one range cut into pieces), against the update that walks all samples (a per-shard
# view in between keeps it to that).  The pieces lie in the per-shard gradient buffer: a view after the update forms
# the shards' gradients there again.  Dense update on the launch stream (1.4 M parameters) and beside it (2.1 M).
@pytest.mark.parametrize("hidden", [(1288, 1032), (1288, 1544)], ids=["launch-stream", "beside"])
@pytest.mark.parametrize("sizes", [(1500, 2700, 1100, 3700), (2300,) * 4], ids=["unequal", "equal"])
def test_weight_gradient_pieces(sizes, hidden):
    import torch
    import paper_2404_09679_amd as A
    from gpu_helpers import GpuRun
    from test_gpu_parity import assert_close, make_inputs
    cfg = _config(f"pieces-{sizes[0]}", 700 + sizes[0], num_fields=3, layer_sizes=hidden, shard_sizes=sizes)
    tables, state, flat, fstate, batch = make_inputs(cfg, nonzero_state=True)
    got, grads = [], []
    for view, profile in ((False, False), (True, False), (False, True), (True, True)):
        run = GpuRun(cfg, tables, flat, state, fstate)
        if profile:
            run.ctx.profile(1)
        run.set_batch(batch)
        run.ctx.assign_shard(batch.batch, len(sizes), sizes=sizes)
        run.ctx.worker_step_all(torch.zeros(len(sizes), device="cuda:0"))
        viewed = [run.ctx.view_shard_grads(k)[0] for k in range(len(sizes))] if view else None
        run.ctx.aggregate()
        run.ctx.apply_update()
        if profile:   # which way the update went
            torch.cuda.synchronize()
            n = {name: run.ctx.profile_read(i)[0] for i, name in enumerate(A.kernel_names())}
            assert (n["gemm_wgrad"], n["dense_adagrad"], n["wgrad_adagrad"]) == ((1, 0, 1) if view else (1, 1, 0))
            continue
        after = viewed if view else [run.ctx.view_shard_grads(k)[0] for k in range(len(sizes))]
        torch.cuda.synchronize()
        grads.append([g.cpu().numpy().copy() for g in after])
        run.ctx.worker_step_all(torch.zeros(len(sizes), device="cuda:0"))   # (from the updated bf16 copies)
        torch.cuda.synchronize()
        got.append((run.params.cpu().numpy().copy(), run.pstate.cpu().numpy().copy(), run.ctx.view_pooled(0).float().cpu().numpy().copy(),
                    run.ctx.view_shard_grads(1)[1].cpu().numpy().copy()))
    for k, (a, b) in enumerate(zip(*grads)):
        assert np.array_equal(a, b), f"gradients of shard {k} viewed after the update"
    # sums over up to 9200 products of fp32, in another order: 1e-6 of their size
    for a, b, what in zip(got[0], got[1], ("MLP parameters", "MLP accumulators", "pooled input", "input gradient")):
        if what == "input gradient":   # (bf16 weights one rounding apart here and there)
            assert np.linalg.norm(a - b) <= 2.0 ** -8 * np.linalg.norm(b), what
        else:
            assert_close(a, b, 1e-6, what, 1e-5)


# Windows of fields that follow one another at any place: one window (no slot for partial sums), exactly one, one lookup
# more, several; hot rows, so that runs cross the windows wherever there are several.
@pytest.mark.parametrize("rows", [2, 40])
def test_window_slots_of_neighbouring_fields(rows, monkeypatch):
    sizes = [0, 1, 257, 128, 300, 255, 256, 513, 127, 512, 511, 129, 258, 2049, 3, 1025]
    B, F = 100, len(sizes)
    cfg = _config(f"slots-{rows}", 650 + rows, num_fields=F, rows_per_field=rows, dim=8, layer_sizes=(8,), gemm_dtype="f32",
                  shard_sizes=(30, 0, 50, 20), max_bag=21, min_bag=0)
    rng = np.random.default_rng(11 + rows)
    _plant(monkeypatch, [rng.integers(0, rows, n) for n in sizes], B,
           lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, mask=(1, 1, 0, 1), nonzero_state=True)


# bf16 products without a hidden layer: the last layer's gradient is formed inside the update as well, or by the step;
# from sums over tiles of samples, or from the samples where most shards hold one
@pytest.mark.parametrize("sizes", [(16, 1, 0, 33, 200), (1,) * 30 + (0, 3) + (1,) * 20 + (2,)], ids=["tiles", "samples"])
@pytest.mark.parametrize("kw", [{}, {"eager": True}, {"streams": False}, {"static": True}], ids=["update", "step", "one-stream", "static"])
def test_bf16_model_without_hidden_layer(kw, sizes):
    import torch
    from gpu_helpers import GpuRun
    from helpers import flat_layers, oracle_iteration, rel_err
    from test_gpu_parity import make_inputs
    cfg = _config("no-hidden-bf16", 668, layer_sizes=(), shard_sizes=sizes)
    check_iteration(cfg, cfg.shard_sizes, tol=TOLBF, bf16_gemm_oracle=True, batched=True, nonzero_state=True)
    tables, state, flat, fstate, batch = make_inputs(cfg, nonzero_state=True)
    _, _, _, upd = oracle_iteration(cfg, tables, state, flat, fstate, batch, cfg.shard_sizes, bf16_gemm=True)
    run = GpuRun(cfg, tables, flat, state, fstate, **kw)
    run.set_batch(batch)
    run.ctx.assign_shard(batch.batch, len(sizes), sizes=sizes)
    run.ctx.worker_step_all(torch.zeros(len(sizes), device="cuda:0"))
    run.ctx.aggregate()
    run.ctx.apply_update()
    torch.cuda.synchronize()
    assert rel_err(run.params.cpu().numpy() - flat, flat_layers(cfg, upd.layers) - flat)[0] <= TOLBF


# No hidden layer: sums over tiles of samples, or per sample where those would need memory of their own (few lookups, many
# dense features); shards of less, exactly and more than a tile
@pytest.mark.parametrize("fields,num_dense,max_bag", [(3, 2, 5), (1, 700, 1)])
def test_f32_model_without_hidden_layer(fields, num_dense, max_bag):
    cfg = _config(f"no-hidden-{fields}", 660 + fields, num_fields=fields, rows_per_field=500, dim=4, num_dense=num_dense, layer_sizes=(),
                  gemm_dtype="f32", shard_sizes=(16, 1, 0, 33, 200), max_bag=max_bag, min_bag=0)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, mask=(1, 1, 1, 0, 1), nonzero_state=True)


# fp32 models: the gradient of the last hidden layer takes the activation's place; widths around the 512 columns that a
# wavefront keeps at once
@pytest.mark.parametrize("width", [1, 63, 512, 513, 1300])
def test_f32_last_hidden_layer(width):
    cfg = _config(f"last-hidden-{width}", 670, layer_sizes=(24, width), gemm_dtype="f32", shard_sizes=(16, 3, 0, 37))
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)


def test_bf16_products_of_rows_beyond_32_bit_offsets():
    """34.1 million dense features: 64 samples of the weight gradient's tile span more than 4 GiB.  Against the same
    products in torch, formed from the library's own pooled input (the hidden layer is small)."""
    import torch
    import paper_2404_09679_amd as A
    nd, B, N = 34_100_003, 70, 8
    cfg = _config("far", 690, num_fields=1, rows_per_field=50, dim=8, num_dense=nd, layer_sizes=(N,), shard_sizes=(B,))
    width = cfg.layer_sizes[0]
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(5)
    params = torch.randn(width * N + N + N + 1, generator=g, device=dev) * 2e-4
    W1 = params[width * N + N:width * N + 2 * N]
    W1.copy_(torch.tensor([1.0, -1.0] * 4, device=dev))
    pstate = torch.ones_like(params)
    tables = torch.randn((50, 8), generator=g, device=dev)
    dense = torch.randn((B, nd), generator=g, device=dev)
    labels = (torch.rand(B, generator=g, device=dev) < 0.5).float()
    ids = torch.randint(0, 50, (B,), generator=g, device=dev, dtype=torch.int32)
    ctx = A.Context(A.model_from_config(cfg, max_nnz=B))
    ctx.bind(tables, torch.ones_like(tables), params, pstate)
    ctx.set_batch(ids, [0, B], torch.arange(B + 1, dtype=torch.int32, device=dev).reshape(1, -1), dense, labels)
    ctx.assign_shard(B, 1)
    loss = torch.zeros(1, device=dev)
    ctx.worker_step_all(loss)
    got, dx = ctx.view_shard_grads(0)
    torch.cuda.synchronize()
    x = ctx.view_pooled(0)
    z = params[width * N:width * N + N].double().expand(B, N).clone()
    step = 1 << 20
    for c in range(0, width, step):
        e = min(width, c + step)
        z += (x[:, c:e].float() @ params[c * N:e * N].reshape(-1, N).bfloat16().float()).double()
    h = z.clamp(min=0).float().bfloat16().double()
    logit = h @ W1.double() + params[-1].double()
    want_loss = torch.nn.functional.binary_cross_entropy_with_logits(logit, labels.double())
    assert abs(loss.item() - want_loss.item()) <= 2e-2 * want_loss.item()
    dh = ((torch.sigmoid(logit) - labels.double()) / B)[:, None] * W1.double() * (h > 0)
    dh = dh.float().bfloat16().float()
    num = den = 0.0
    for c in range(0, width, step):
        e = min(width, c + step)
        want = x[:, c:e].float().T @ dh
        num += float(((got[c * N:e * N].reshape(-1, N) - want) ** 2).sum())
        den += float((want ** 2).sum())
    assert num <= (TOLBF * TOLBF) * den
    want = dh @ params[:8 * N].reshape(8, N).bfloat16().float().T
    assert float((dx - want).norm()) <= TOLBF * float(want.norm())


# Windows inside one run (256 sorted lookups, 512 from four million of them on: see test_sort_ahead_of_the_gather): summed
# by every wavefront for itself, neighbours of one sample as one.  A field of one row only, one window and several; bags that
# repeat a row 1 .. 300 times; the first window of a run, one in its middle, its last, and a run of exactly one window.
@pytest.mark.parametrize("dim,pooling,table,state", [(4, "sum", "f32", "elementwise"), (32, "mean", "f32", "rowwise"),
                                                     (64, "sum", "bf16", "rowwise"), (256, "mean", "f32", "elementwise")])
def test_windows_inside_one_run(dim, pooling, table, state, monkeypatch):
    runs = [[256], [512], [700], [256, 256, 512], [100, 156, 256, 900], [255, 1, 1500, 36, 1, 256]]
    B = 70
    cfg = _config(f"inside-{dim}", 680 + dim, num_fields=len(runs), rows_per_field=9, dim=dim, table_dtype=table, adagrad_state=state,
                  layer_sizes=(8,), gemm_dtype="f32", shard_sizes=(30, 1, 39), max_bag=300, pooling=pooling)
    rng = np.random.default_rng(17 + dim)
    ids, offsets = [], []
    for lengths in runs:   # a run's lookups, dealt to samples in lumps: the bags of a sample hold lumps of several rows
        bags = [[] for _ in range(B)]
        for row, n in enumerate(lengths):
            while n > 0:
                lump = min(n, int(rng.choice([1, 2, 5, 64, 65, 300])))
                bags[rng.integers(0, B)] += [row] * lump
                n -= lump
        ids.append(np.array(sum(bags, []), dtype=np.int32))
        offsets.append(np.cumsum([0] + [len(b) for b in bags]))
    _plant(monkeypatch, ids, B, lambda f, n: offsets[f])
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)


# The row update takes square root and quotient by a short way where the accumulators lie between 2^-90 and 2^90, by the
# general one elsewhere: accumulators of both kinds, and with them NaN and infinities, side by side in a wavefront.
@pytest.mark.parametrize("dim,state", [(4, "elementwise"), (16, "rowwise"), (128, "elementwise")])
def test_row_update_over_the_range_of_accumulators(dim, state):
    import torch
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    cfg = _config(f"range-{dim}", 685 + dim, num_fields=1, rows_per_field=40, dim=dim, layer_sizes=(8,), gemm_dtype="f32", shard_sizes=(50,),
                  eps=1e-8, max_bag=2)
    cfg = dataclasses.replace(cfg, adagrad_state=state)
    values = np.array([0.0, 1e-40, 1e-30, 2.0 ** -90, 1e-12, 1e-4, 1.0, 1e20, 1.2e27, 2.0 ** 90, 1e38, np.inf, np.nan], dtype=np.float32)
    tables, acc, flat, fstate, batch = make_inputs(cfg, True)
    shape = acc.shape
    acc = np.resize(values, acc.size).reshape(shape)
    run = GpuRun(cfg, tables, flat, acc, fstate)
    run.set_batch(batch)
    run.iteration(cfg.shard_sizes, batched=True)
    u, _, _, G = run.coalesced[0]
    with np.errstate(all="ignore"):
        g, S, p = G.astype(np.float64), acc[u].astype(np.float64), tables[u].astype(np.float64)
        S = S + (g * g if state == "elementwise" else np.mean(g * g, axis=1))
        step = cfg.lr * g / (np.sqrt(S if state == "elementwise" else S[:, None]) + cfg.eps)
    got_s, got_p = run.state.cpu().numpy()[u], run.tables.cpu().numpy()[u]
    assert np.array_equal(np.isnan(got_s), np.isnan(S)) and np.array_equal(np.isinf(got_s), np.isinf(S))
    fine = np.isfinite(S)
    assert np.all(np.abs(got_s[fine] - S[fine]) <= 1e-6 * S[fine] + 1e-44)
    assert np.array_equal(np.isnan(got_p), np.isnan(step))
    ok = ~np.isnan(step)
    # a few roundings of the step, and that of the stored parameter
    assert np.all(np.abs(got_p[ok] - (p - step)[ok]) <= 1e-6 * np.abs(step[ok]) + 2.0 ** -23 * np.abs(p[ok]))


# The same to the bit: gradients and accumulators over the whole range, each row one lookup's (a table of zeros shows the quotient itself).
@pytest.mark.parametrize("dim,state,lr", [(128, "elementwise", 0.01), (4, "elementwise", 2.0 ** 31), (64, "rowwise", 1.0), (256, "rowwise", 2.0 ** -20)])
def test_row_update_rounds_as_a_division_does(dim, state, lr):
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    F, B = 4, 500
    cfg = _config(f"rounds-{dim}", 690 + dim, num_fields=F, rows_per_field=B, dim=dim, layer_sizes=(), gemm_dtype="f32", shard_sizes=(200, 300),
                  adagrad_state=state, max_bag=1, lr=lr)
    rng = np.random.default_rng(dim)
    _, acc, flat, fstate, batch = make_inputs(cfg)
    span = 2.0 ** rng.uniform(-135, 40, flat.shape)   # (dX = dz w, dz about 1e-3)
    flat = (span * rng.choice([-1.0, 1.0], flat.shape) * (rng.random(flat.shape) > 0.05)).astype(np.float32)
    flat[1::5] *= np.float32(2.0 ** -115) / np.abs(flat[1::5]).clip(2.0 ** -135)   # (some of them tiny whatever the width)
    flat[-1] = 0.0
    acc = (2.0 ** rng.uniform(-85, 85, acc.shape)).astype(np.float32)
    acc[::7] = (2.0 ** rng.uniform(-140, 120, acc[::7].shape)).astype(np.float32)
    ids = np.concatenate([rng.permutation(B) for _ in range(F)]).astype(np.int32)
    batch = dataclasses.replace(batch, ids=ids, offsets=np.tile(np.arange(B + 1, dtype=np.int32), (F, 1)), field_ptr=np.arange(F + 1, dtype=np.int64) * B,
                                dense=np.zeros_like(batch.dense))
    run = GpuRun(cfg, np.zeros((F * B, dim), np.float32), flat, acc, fstate, max_batch=B, max_nnz=F * B)
    run.set_batch(batch)
    run.iteration(cfg.shard_sizes, batched=True)
    got, S = run.tables.cpu().numpy(), run.state.cpu().numpy()
    tiny = 0
    with np.errstate(all="ignore"):
        for f in range(F):
            u, _, _, G = run.coalesced[f]
            rows = f * B + u
            tiny += np.sum((np.abs(G) > 0) & (np.abs(G) < 2.0 ** -110))
            den = np.sqrt(S[rows] if state == "elementwise" else S[rows][:, None]) + np.float32(cfg.eps)
            want = np.float32(0) - np.float32(lr) * G / den
            assert den.dtype == want.dtype == np.float32
            assert np.array_equal(got[rows], want)
    assert tiny > 100


# The gather hands the 64 samples of a block out by the number of iterations their bags take (fifteen and more are one class):
# equal bags, bags of every length up to 300, empty ones, blocks that end inside.  Rows of 4, 8 and 16 pieces of 16 bytes.  (Rows of 4
# pieces, and batches of short bags, as they come.)
@pytest.mark.parametrize("bags", ["short", "long"])
@pytest.mark.parametrize("dim,table,pooling", [(16, "f32", "sum"), (32, "f32", "mean"), (128, "bf16", "sum"), (32, "bf16", "mean")])
def test_gather_of_bags_of_many_lengths(dim, table, pooling, bags, monkeypatch):
    F, B = 40, 1700   # (enough blocks that they take 64 samples each)
    assert F * (-(-B // 64)) >= 1024 and B % 64
    cfg = _config(f"bags-{dim}", 690 + dim, num_fields=F, rows_per_field=300, dim=dim, table_dtype=table, adagrad_state="rowwise", layer_sizes=(8,),
                  gemm_dtype="f32", shard_sizes=(700, 1, 999), max_bag=300, pooling=pooling)
    rng = np.random.default_rng(dim)
    lengths = [rng.integers(0, 3 if bags == "short" else 20, B) for _ in range(F)]
    lengths[0] = np.full(B, 7)
    lengths[1] = rng.integers(0, 130, B)
    lengths[2] = np.where(np.arange(B) % 64 == 17, 300, 0)
    lengths[3] = np.arange(B) % 66
    lengths[4] = (np.arange(B) == B - 1).astype(int)
    assert (sum(n.sum() for n in lengths) >= 8 * F * B) == (bags == "long")
    ids = [rng.integers(0, 300, n.sum()) for n in lengths]
    _plant(monkeypatch, ids, B, lambda f, n: np.concatenate([[0], np.cumsum(lengths[f])]))
    # (accumulators from zero: with others, of about 1e-4, a step is about 1e-4 or less, and rounding the stored parameter of about
    # 0.05 to fp32, 2^-25 * 0.05 = 1.5e-9, is 1.5e-5 of it: more than the 1e-5 that steps are compared to)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True)


# Fields that fit one window of the reduction: the longest of 1024 or 2048 lookups, one fewer or more; one long run, runs
# around the lengths that are cut into pieces, single lookups.  Rows of 128 columns keep the windows of 256.
@pytest.mark.parametrize("most", [1, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("dim,table,state,pooling", [(4, "f32", "rowwise", "sum"), (16, "f32", "elementwise", "mean"), (64, "f32", "elementwise", "sum"),
                                                     (64, "bf16", "rowwise", "mean"), (128, "f32", "elementwise", "sum")])
def test_windows_of_whole_fields(most, dim, table, state, pooling, monkeypatch):
    sizes = [most, max(most - 1, 1), most // 2 + 1, 1, most]
    B = 90
    cfg = _config(f"whole-{dim}", 720 + dim, num_fields=len(sizes), rows_per_field=2300, dim=dim, table_dtype=table, adagrad_state=state, layer_sizes=(8,),
                  gemm_dtype="f32", shard_sizes=(30, 0, 59, 1), max_bag=60, min_bag=0, pooling=pooling)
    rng = np.random.default_rng(most + dim)
    lengths = [700, 1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 48, 250]
    ids = []
    for f, n in enumerate(sizes):
        rows = np.repeat(np.arange(len(lengths)) * 170, lengths)[:n] if f < 4 else np.full(n, 2299)   # (the last field: one run)
        rows = np.concatenate([rows, rng.permutation(2300)[:n - len(rows)]])
        ids.append(rng.permutation(rows))
    _plant(monkeypatch, ids, B, lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    # (accumulators from zero: see test_sort_over_many_blocks)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True)


# fp32 models of a batched step: the sort of fields that fit a block in the weight-gradient launch, tiles of 32 rows and columns
# (many shards) and of 16, each size of the sort; an empty field, an empty shard, blocks of four tiles that are not all there
@pytest.mark.parametrize("most", [2048, 4096, 8192, 16384])
@pytest.mark.parametrize("hidden,shards", [((264, 136), (90, 1, 0, 200, 9, 50)), ((40, 24), (341, 9))], ids=["tiles-32", "tiles-16"])
def test_sort_beside_the_weight_gradients(most, hidden, shards, monkeypatch):
    sizes = [most, most // 2 + 1, 0, 1]
    B = sum(shards)
    cfg = _config(f"beside-{most}", 760, num_fields=len(sizes), rows_per_field=3000, dim=8, layer_sizes=hidden, gemm_dtype="f32", shard_sizes=shards,
                  max_bag=most // 300 + 2, min_bag=0)
    rng = np.random.default_rng(most)
    ids = [rng.integers(0, 3000, n) // rng.integers(1, 40, n) for n in sizes]
    _plant(monkeypatch, ids, B, lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    # (accumulators from zero: see test_sort_over_many_blocks)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True)


# Many gradient tiles and short fields keep the sort to a launch of its own, ahead of the reduction; few tiles or longer fields do not.
# Class counts say which way a step went.
@pytest.mark.parametrize("hidden,shards,most,launches", [((1024, 512), (8,) * 12, 300, 1), ((1024, 512), (24,) * 4, 300, 0), ((1024, 512), (8,) * 12, 16_384, 0),
                                                         ((64, 32), (24,) * 4, 300, 0), ((64, 32), (24,) * 4, 16_385, 6)])
def test_where_an_fp32_step_sorts(hidden, shards, most, launches, monkeypatch):
    import torch
    import paper_2404_09679_amd as A
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    B = sum(shards)
    cfg = _config(f"where-{most}", 780, layer_sizes=hidden, gemm_dtype="f32", shard_sizes=shards, max_bag=most // 90 + 2, rows_per_field=200_000)
    rng = np.random.default_rng(most)
    _plant(monkeypatch, [rng.integers(0, 200_000, n) for n in (most, 5, most // 2)], B,
           lambda f, n: np.concatenate([[0], np.sort(rng.integers(0, n + 1, B - 1)), [n]]))
    tables, state, flat, fstate, batch = make_inputs(cfg)
    run = GpuRun(cfg, tables, flat, state, fstate, streams=False)
    run.ctx.profile(1)
    run.set_batch(batch)
    run.ctx.assign_shard(B, len(shards), sizes=shards)
    run.ctx.worker_step_all(torch.zeros(len(shards), device="cuda:0"))
    run.ctx.aggregate()
    run.ctx.apply_update()
    torch.cuda.synchronize()
    n = {name: run.ctx.profile_read(i)[0] for i, name in enumerate(A.kernel_names())}
    assert n["gemm_wgrad"] == 1 and n["sort_hist"] + n["sort_scan"] + n["sort_scatter"] == launches
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True)


# The loss kernel adds a logit's products in one order, whatever the type, the width and the way the columns are loaded: 64 chains
# of every 64th column, then the chains in halves.  (Another order moves logits by their last bit, and with them the entries of
# bf16 gradients that lie between two neighbours.)  A shard's loss shows the logit of one of its samples bit for bit: at a label of 0 and
# z >= 32 the loss is z (what is added to it is below 2e-14), at z = -1000 it is 0, and lengths are powers of two.
@pytest.mark.parametrize("gemm,width,hidden", [("f32", 13, False), ("f32", 256, False), ("f32", 704, False), ("f32", 131, True), ("f32", 128, True),
                                               ("bf16", 264, False), ("bf16", 66, False), ("bf16", 8, True), ("bf16", 72, True),
                                               ("bf16", 256, True), ("bf16", 512, True), ("bf16", 1096, True)])
def test_order_of_a_logit(gemm, width, hidden):
    import torch
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    sizes = (16,) * 16 + (1, 2, 8)
    shown = [i for i in range(16)] + [0, 1, 5]   # whose logit is the shard's loss
    num_dense = width if hidden else width - 4   # (a pooled field of four columns ahead, all bags empty)
    cfg = _config(f"logit-{gemm}-{width}", 770, num_fields=1, rows_per_field=8, dim=4, num_dense=num_dense, layer_sizes=(width,) if hidden else (),
                  gemm_dtype=gemm, shard_sizes=sizes, min_bag=0, max_bag=1)
    B, K = sum(sizes), len(sizes)
    rng = np.random.default_rng(width)
    kill, first = num_dense // 2, np.cumsum((0,) + sizes)
    dense = np.zeros((B, num_dense), dtype=np.float32)
    dense[:, kill] = 1.0
    for k in range(K):   # (bf16 values: a hidden layer that passes them on does so exactly)
        dense[first[k] + shown[k]] = rng.integers(64, 128, num_dense) / 64.0
        dense[first[k] + shown[k], kill] = 0.0
    w = rng.uniform(1.0, 16.0, width).astype(np.float32)
    w[(0 if hidden else 4) + kill] = -1000.0
    bias = np.float32(0.37)
    parts = [np.concatenate([np.zeros((4, width)), np.eye(width)]).reshape(-1), np.zeros(width)] if hidden else []
    flat = np.concatenate(parts + [w, [bias]]).astype(np.float32)
    tables, state, _, _, batch = make_inputs(cfg)
    batch = dataclasses.replace(batch, ids=np.zeros(0, np.int32), offsets=np.zeros((1, B + 1), np.int32), field_ptr=np.zeros(2, np.int64),
                                dense=dense, labels=np.zeros(B, np.float32))
    run = GpuRun(cfg, tables, flat, state, max_batch=B, max_nnz=1)
    run.set_batch(batch)
    run.ctx.assign_shard(B, K, sizes=sizes)
    loss = torch.zeros(K, device="cuda:0")
    run.ctx.worker_step_all(loss)
    torch.cuda.synchronize()
    h = dense[[first[k] + shown[k] for k in range(K)]]
    if not hidden:
        h = np.concatenate([np.zeros((K, 4), np.float32), h], axis=1)
    chains = np.zeros((K, 64), np.float32)
    for j0 in range(0, width, 64):   # (products of 8 and 24 bits, added to 24: exact in 64-bit floats, rounded once)
        n = min(64, width - j0)
        chains[:, :n] = (h[:, j0:j0 + n].astype(np.float64) * w[j0:j0 + n] + chains[:, :n]).astype(np.float32)
    for o in (32, 16, 8, 4, 2, 1):
        chains = chains[:, :o] + chains[:, o:2 * o]
    z = chains[:, 0] + bias
    assert np.all(z >= 32)
    assert np.array_equal(loss.cpu().numpy() * np.array(sizes, np.float32), z)


# The gradient of the pooled input beside the weight gradients: the bits of a launch of its own (made while a class is timed), for fp32
# tiles of 16 and of 32 rows and columns of both products, rows at any place and too short for that (a launch of its own either way), and bf16
# tiles of 32 and of 64, and from 200 tiles of 128 on (its own); an empty shard, remainders of tiles and of blocks.
@pytest.mark.parametrize("gemm,sizes,hidden,num_dense", [("f32", (90, 1, 0, 200, 9, 50), (264, 136), 3), ("f32", (17,), (40, 24), 0),
                                                         ("f32", (1500, 40), (101,), 5), ("f32", (33, 31), (3,), 1), ("f32", (4100,), (72, 40), 2), ("f32", (900,) * 4, (256, 128), 7),
                                                         ("bf16", (5, 0, 60), (264, 72), 13), ("bf16", (700, 9), (264, 72), 0),
                                                         ("bf16", (3300, 0, 4100), (136,), 13)])
def test_input_gradient_beside_the_weight_gradients(gemm, sizes, hidden, num_dense):
    import torch
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    cfg = _config(f"joined-{gemm}-{sum(sizes)}", 790, num_fields=12, dim=32, layer_sizes=hidden, num_dense=num_dense, gemm_dtype=gemm, shard_sizes=sizes,
                  table_dtype="f32")
    tables, state, flat, fstate, batch = make_inputs(cfg)
    out = []
    for mode in (0, 1):
        run = GpuRun(cfg, tables, flat, state, fstate, streams=False, eager=True)
        run.ctx.profile(mode)
        run.set_batch(batch)
        run.ctx.assign_shard(sum(sizes), len(sizes), sizes=sizes)
        loss = torch.full((len(sizes),), -1.0, device="cuda:0")
        run.ctx.worker_step_all(loss)
        torch.cuda.synchronize()
        views = [t.cpu().numpy().copy() for k in range(len(sizes)) for t in run.ctx.view_shard_grads(k)]
        out.append([loss.cpu().numpy()] + views)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    if gemm == "f32":
        check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True)


# The dense update of an fp32 model in blocks of the sparse update's launch: the bits of a launch of its own (made while a class is timed), for
# windows of 256 lookups and of whole fields, fewer parameters than a block and more than many, a shard left out that never stepped, and no
# lookups at all (a launch of its own either way).
@pytest.mark.parametrize("hidden,fields,max_bag,mask", [((), 1, 1, None), ((40, 24), 3, 3, (1, 0, 1)), ((40, 24), 2, 90, None), ((264, 136), 12, 30, (1, 0, 1)),
                                                        ((72,), 3, 0, None)])
def test_dense_update_beside_the_sparse_one(hidden, fields, max_bag, mask):
    import torch
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    sizes = (70, 33, 6)
    cfg = _config(f"dense-{max_bag}", 800, num_fields=fields, layer_sizes=hidden, gemm_dtype="f32", shard_sizes=sizes, max_bag=max(max_bag, 1),
                  min_bag=0 if max_bag == 0 else 1)
    tables, state, flat, fstate, batch = make_inputs(cfg, True)
    if max_bag == 0:
        batch = dataclasses.replace(batch, ids=np.zeros(0, np.int32), offsets=np.zeros((fields, sum(sizes) + 1), np.int32),
                                    field_ptr=np.zeros(fields + 1, np.int64))
    out = []
    for mode in (0, 1):
        run = GpuRun(cfg, tables, flat, state, fstate)
        run.ctx.profile(mode)
        run.set_batch(batch)
        run.ctx.assign_shard(sum(sizes), len(sizes), sizes=sizes)
        loss = torch.zeros(len(sizes), device="cuda:0")
        for k in range(len(sizes)):
            if mask is None or mask[k]:
                run.ctx.worker_step(k, loss[k:k + 1])
        run.ctx.aggregate(mask)
        run.ctx.apply_update()
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (run.params, run.pstate, run.tables, run.state, loss)])
    assert not np.array_equal(out[0][0], flat)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
