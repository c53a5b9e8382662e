"""The order of the calls and the streams they go to: captured iterations, worker steps on streams of their
own, views between and after the calls, options changed on the way.  The same work in the plainest order
(one stream, no view, nothing captured) is the reference; sums are formed in the same order, so results are equal bit
for bit unless stated."""
import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu

# bf16 products; 52 000 lookups and 0.09 M parameters (dense update on the launch stream) or 2.3 M (on a stream of its own)
SMALL_BF = wl.RankingConfig("order-small", 5, 20_000, 32, "f32", "elementwise", 13, (173, 256, 128, 64, 1), "bf16",
                            20, 1.1, (300, 37, 0, 663), wl.SEED0 + 801)
WIDE_BF = wl.scaled(SMALL_BF, name="order-wide", layer_sizes=(173, 2048, 1024, 1))


def start(cfg, **kw):
    from gpu_helpers import GpuRun
    from test_gpu_parity import make_inputs
    tables, state, flat, fstate, batch = make_inputs(cfg, nonzero_state=True)
    run = GpuRun(cfg, tables, flat, state, fstate, max_batch=batch.batch, max_shards=len(cfg.shard_sizes),
                 max_nnz=int(batch.field_ptr[-1]), **kw)
    run.set_batch(batch)
    run.ctx.assign_shard(batch.batch, len(cfg.shard_sizes), sizes=cfg.shard_sizes)
    run.loss = torch.zeros(len(cfg.shard_sizes), device="cuda:0")
    torch.cuda.synchronize()
    return run


def step(run):
    run.ctx.worker_step_all(run.loss)
    run.ctx.aggregate()
    run.ctx.apply_update()


def weights(run):
    torch.cuda.synchronize()
    return [t.float().cpu().numpy().copy() for t in (run.loss, run.params, run.pstate, run.tables, run.state)]


def assert_same(a, b, what):
    for x, y, name in zip(a, b, ("losses", "MLP parameters", "MLP accumulators", "tables", "accumulators")):
        assert np.array_equal(x, y), f"{what}: {name}"


@pytest.mark.parametrize("cfg,streams", [(SMALL_BF, False), (WIDE_BF, False), (WIDE_BF, True)],
                         ids=["small-one-stream", "wide-one-stream", "wide"])
def test_replays_of_a_captured_iteration(cfg, streams):
    """Every replay reads the weights that the one before wrote, the bf16 copy of the first layer's among them, also with
    iterations outside the graph in between."""
    ref, run = start(cfg, streams=streams), start(cfg, streams=streams)
    step(ref)
    step(run)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(run)
    for i in range(4):
        step(ref)
        graph.replay()
        assert_same(weights(run), weights(ref), f"replay {i}")
        for k in (1, 3):
            for a, b in zip(run.ctx.view_shard_grads(k), ref.ctx.view_shard_grads(k)):
                torch.cuda.synchronize()
                assert torch.equal(a, b), f"gradients of shard {k}, replay {i}"
        if i == 1:
            step(ref)
            step(run)
            assert_same(weights(run), weights(ref), "iteration between the replays")


def on_streams_of_their_own(run, delayed=()):
    """One worker_step per shard, each on its own stream behind everything enqueued so far (`delayed`: these
    start late); the current stream continues behind all of them."""
    main = torch.cuda.current_stream()
    ready = torch.cuda.Event()
    ready.record(main)
    for k in range(len(run.cfg.shard_sizes)):
        s = torch.cuda.Stream()
        s.wait_event(ready)
        with torch.cuda.stream(s):
            if k in delayed:
                torch.cuda._sleep(4_000_000)   # about two milliseconds
            run.ctx.worker_step(k, run.loss[k:k + 1])
        main.wait_stream(s)


@pytest.mark.parametrize("cfg", [wl.scaled(SMALL_BF, name="order-f32", gemm_dtype="f32"), SMALL_BF,
                                 wl.scaled(SMALL_BF, name="order-one-layer", layer_sizes=(173, 1))], ids=lambda c: c.name)
def test_losses_of_worker_steps_on_different_streams(cfg):
    """What a step leaves for the launch that adds up its losses is not overwritten by another worker's step."""
    ref, run = start(cfg), start(cfg)
    for k in range(len(cfg.shard_sizes)):
        ref.ctx.worker_step(k, ref.loss[k:k + 1])
    torch.cuda.synchronize()
    for _ in range(8):
        run.loss.fill_(-1.0)
        on_streams_of_their_own(run)
        torch.cuda.synchronize()
        assert torch.equal(run.loss, ref.loss)


@pytest.mark.parametrize("view", [False, True], ids=["update", "view"])
@pytest.mark.parametrize("cfg", [SMALL_BF, WIDE_BF], ids=lambda c: c.name)
def test_update_waits_for_worker_steps_on_different_streams(cfg, view):
    """The weight gradients are formed behind all workers' steps, not only behind the one enqueued last."""
    ref, run = start(cfg), start(cfg)
    for _ in range(2):
        for k in range(len(cfg.shard_sizes)):
            ref.ctx.worker_step(k, ref.loss[k:k + 1])
        on_streams_of_their_own(run, delayed=(0, 1))
        if view:
            a, b = run.ctx.view_shard_grads(0)[0], ref.ctx.view_shard_grads(0)[0]
            torch.cuda.synchronize()
            assert torch.equal(a, b)
        for r in (ref, run):
            r.ctx.aggregate()
            r.ctx.apply_update()
        assert_same(weights(run), weights(ref), "update")


# enough samples per shard that the update forms the weight gradients in pieces, in the per-shard gradient buffer
PIECES = wl.RankingConfig("order-pieces", 3, 2000, 16, "f32", "elementwise", 5, (53, 1288, 1032, 1), "bf16", 3, 1.1,
                          (1500, 2700, 1100, 3700), wl.SEED0 + 810)


def test_viewed_gradients_stay_through_the_update():
    """A shard's gradients viewed before the other workers' steps are the same after the update, which has to
    form all weight gradients itself then."""
    run = start(PIECES)
    run.ctx.worker_step(0, run.loss[:1])
    dense, dx = run.ctx.view_shard_grads(0)
    torch.cuda.synchronize()
    before = dense.clone(), dx.clone()
    for k in range(1, 4):
        run.ctx.worker_step(k, run.loss[k:k + 1])
    run.ctx.aggregate()
    run.ctx.apply_update()
    torch.cuda.synchronize()
    assert torch.equal(dense, before[0]) and torch.equal(dx, before[1])


@pytest.mark.parametrize("first,then", [(False, True), (True, False)], ids=["deferred-then-eager", "eager-then-deferred"])
def test_weight_gradient_option_changed_between_worker_steps(first, then):
    """Whichever steps left their weight gradients to the update, all of them are in it, and in the views."""
    ref, run = start(SMALL_BF), start(SMALL_BF)
    for k in range(4):
        ref.ctx.worker_step(k, ref.loss[k:k + 1])
        run.ctx.set_eager_weight_gradients(first if k < 2 else then)
        run.ctx.worker_step(k, run.loss[k:k + 1])
    for r in (ref, run):
        r.ctx.aggregate()
        r.ctx.apply_update()
    assert_same(weights(run), weights(ref), "update")
    for k in (0, 1, 3):
        a, b = run.ctx.view_shard_grads(k)[0], ref.ctx.view_shard_grads(k)[0]
        torch.cuda.synchronize()
        assert torch.equal(a, b), f"shard {k}"


# (the last three: 100 000 lookups and more, and few blocks over many samples, a large model on few samples, and pieces)
@pytest.mark.parametrize("cfg", [WIDE_BF, wl.scaled(WIDE_BF, name="order-equal", shard_sizes=(250,) * 4),
                                 wl.scaled(PIECES, name="order-pieces-wide", layer_sizes=(53, 1288, 1544, 1)),
                                 wl.scaled(SMALL_BF, name="order-many-samples", shard_sizes=(3000, 37, 0, 5163), max_bag=5),
                                 wl.scaled(SMALL_BF, name="order-large-model", layer_sizes=(173, 1032, 1048, 1), shard_sizes=(700, 37, 0, 2263), max_bag=14),
                                 wl.scaled(SMALL_BF, name="order-pieces-long", layer_sizes=(173, 1288, 1032, 1), shard_sizes=(1750,) * 4, max_bag=6)],
                         ids=lambda c: c.name)
@pytest.mark.parametrize("batched", [True, False], ids=["batched", "by-worker"])
def test_dense_update_beside_the_launch_stream(cfg, batched):
    """Models whose dense update runs beside the input gradient and the sparse update (batched steps; after steps by worker
    once shards are left out), fused with the weight gradients of several ranges or one, or from pieces; no view in
    between that would wait for anything.  Three iterations, the last two on the weights of the ones before."""
    runs = [start(cfg, streams=s) for s in (True, False)]
    K = len(cfg.shard_sizes)
    for _ in range(3):
        for run in runs:
            if batched:
                run.ctx.worker_step_all(run.loss)
                run.ctx.aggregate()
            else:
                for k in range(1, K):
                    run.ctx.worker_step(k, run.loss[k:k + 1])
                run.ctx.aggregate([0] + [1] * (K - 1))
            run.ctx.apply_update()
    assert_same(weights(runs[0]), weights(runs[1]), "three iterations")


# The same with the sort on a stream of its own (105 000 lookups) and, of fp32 models, in the weight-gradient launch
LONG_BF = wl.scaled(WIDE_BF, name="order-long", shard_sizes=(600, 74, 0, 1326))


@pytest.mark.parametrize("cfg,streams", [(LONG_BF, True), (wl.scaled(LONG_BF, name="order-long-f32", gemm_dtype="f32", layer_sizes=(173, 256, 64, 1)), True),
                                         (wl.scaled(SMALL_BF, name="order-f32", gemm_dtype="f32"), True),
                                         (wl.scaled(SMALL_BF, name="order-f32", gemm_dtype="f32"), False)],
                         ids=["sort-beside", "sort-beside-f32", "sort-in-launch", "sort-in-launch-one-stream"])
def test_replays_with_the_sort_elsewhere(cfg, streams):
    assert (len(wl.make_batch(cfg).ids) >= 100_000) == cfg.name.startswith("order-long")
    test_replays_of_a_captured_iteration(cfg, streams)


@pytest.mark.parametrize("cfg", [wl.scaled(SMALL_BF, name="order-f32", gemm_dtype="f32"), LONG_BF], ids=lambda c: c.name)
def test_factors_set_behind_a_batched_step(cfg):
    """The sort of the batched step stays; the weights are the new ones."""
    scale = (0.5, 2.0, 1.0, 1.5)
    early, late = start(cfg), start(cfg)
    early.ctx.set_shard_scale(scale)
    step(early)
    late.ctx.worker_step_all(late.loss)
    late.ctx.set_shard_scale(scale)
    late.ctx.aggregate()
    late.ctx.apply_update()
    assert_same(weights(late), weights(early), cfg.name)


def sorts(run):
    """Launches of the sort (of fields that fit a block) since the last call, apart from those in a weight-gradient launch."""
    import paper_2404_09679_amd as A
    torch.cuda.synchronize()
    return run.ctx.profile_read(A.kernel_names().index("sort_scatter"))[0]


FEW = wl.scaled(SMALL_BF, name="order-few", num_fields=4, layer_sizes=(141, 1024, 256, 1), shard_sizes=(300, 37, 0, 663))


@pytest.mark.parametrize("cfg,ahead", [(FEW, True), (wl.scaled(FEW, layer_sizes=(141, 256, 64, 1)), False),                     # (a short MLP)
                                       (wl.scaled(FEW, max_bag=6), False),                                                      # (short fields)
                                       (wl.scaled(FEW, layer_sizes=(141, 64, 1), shard_sizes=(1500, 1100), max_bag=20), True),  # (100 000 lookups)
                                       (wl.scaled(FEW, gemm_dtype="f32"), False),                                               # (in the weight-gradient launch)
                                       (wl.scaled(FEW, gemm_dtype="f32", layer_sizes=(141, 64, 1), shard_sizes=(8192,), max_bag=3), True),
                                       (wl.scaled(FEW, gemm_dtype="f32", shard_sizes=(850,), max_bag=45), True)],               # (fields too long for that launch)
                         ids=["work", "short-mlp", "short-fields", "many-lookups", "f32-joined", "f32-samples", "f32-long-fields"])
def test_steps_that_sort_ahead(cfg, ahead):
    """Where the sort of a batched step goes to a stream of its own it is enqueued by the step and not by the aggregation; the results are those
    of one stream either way."""
    lookups = np.diff(wl.make_batch(cfg).field_ptr)
    assert lookups.sum() < 100_000 or cfg.layer_sizes == (141, 64, 1)
    run, ref = start(cfg), start(cfg, streams=False)
    run.ctx.profile(1)
    for _ in range(2):
        run.ctx.worker_step_all(run.loss)
        assert (sorts(run) > 0) == ahead
        run.ctx.aggregate()
        run.ctx.apply_update()
        sorts(run)
        step(ref)
    assert_same(weights(run), weights(ref), cfg.name)


def test_steps_whose_sort_nobody_uses():
    """fp32 models sort in the weight-gradient launch of a batched step, but not behind a step whose sort was not used (shards left out,
    gradients only); an aggregation of all shards brings it back.  Results are those of steps that never left it out."""
    cfg = wl.scaled(SMALL_BF, name="order-f32", gemm_dtype="f32")
    run, ref = start(cfg, streams=False), start(cfg, streams=False)
    run.ctx.profile(1)
    mask = [0, 1, 1, 1]
    for i, (use, launches) in enumerate([(None, 0), (mask, 1), (mask, 1), (None, 1), (None, 0), ("step", 0), ("step", 0), (None, 1), (None, 0)]):
        run.ctx.worker_step_all(run.loss)
        if use == "step":
            assert sorts(run) == 0
            continue
        for k in range(4):
            if not use or use[k]:
                ref.ctx.worker_step(k, ref.loss[k:k + 1])
        for r in (run, ref):
            r.ctx.aggregate(use)
            r.ctx.apply_update()
        assert sorts(run) == launches, i
        if not use:   # (of a shard that was left out the steps by worker form no loss)
            assert_same(weights(run), weights(ref), f"iteration {i}")


@pytest.mark.parametrize("graph_of", ["step", "aggregation", "aggregation behind another"])
def test_samples_of_a_large_batch_behind_a_graph(graph_of):
    """A step of more than eight million lookups leaves their sample indices to its sort; an aggregation that sorts anew finds them all the same, also if the
    step is a replay on other bags of the same number of lookups, or if what wrote them is a graph that has not run."""
    import paper_2404_09679_amd as A
    dev, F, rows, B, n = "cuda:0", 3, 5000, 4000, 2_800_000
    cfg = wl.scaled(SMALL_BF, name="order-samples", num_fields=F, rows_per_field=rows, dim=8, num_dense=0, layer_sizes=(24, 16, 1), shard_sizes=(2500, B - 2500))
    g = torch.Generator(device=dev).manual_seed(3)
    ids = torch.empty(F * n, dtype=torch.int32, device=dev)
    offsets = torch.zeros((F, B + 1), dtype=torch.int32, device=dev)

    def draw():
        ids.copy_(torch.randint(0, rows, (F * n,), generator=g, device=dev))
        offsets[:, 1:B] = torch.sort(torch.randint(0, n + 1, (F, B - 1), generator=g, device=dev))[0].int()
        offsets[:, B] = n

    draw()
    tables = torch.randn((F * rows, 8), generator=g, device=dev) * 0.05
    params = torch.randn(24 * 16 + 16 + 17, generator=g, device=dev) * 0.3
    ctx = A.Context(A.model_from_config(cfg, max_batch=B, max_nnz=F * n, max_shards=2))
    ctx.bind(tables, torch.ones_like(tables), params, torch.ones_like(params))
    ctx.set_batch(ids, [f * n for f in range(F + 1)], offsets, None, torch.zeros(B, device=dev))
    ctx.assign_shard(B, 2, sizes=cfg.shard_sizes)
    loss = torch.zeros(2, device=dev)

    def check(mask, below):
        if mask != "replayed":
            ctx.aggregate(mask)
        for f in range(F):
            sample = torch.repeat_interleave(torch.arange(B, device=dev), (offsets[f, 1:] - offsets[f, :-1]).long())
            key, order = torch.sort(ids[f * n:(f + 1) * n][sample < below], stable=True)
            u, so, ss, _ = ctx.view_coalesced(f)
            assert torch.equal(u, torch.unique_consecutive(key)) and torch.equal(ss.long(), sample[sample < below][order]), f

    ctx.worker_step_all(loss)
    check(None, B)
    if graph_of == "aggregation behind another":   # (the indices are there when the graph is made, and not when it is replayed)
        check([1, 0], 2500)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        if graph_of == "step":
            ctx.worker_step_all(loss)
        ctx.aggregate()
    if graph_of != "step":
        check([1, 0], 2500)
    for _ in range(3):
        draw()
        if graph_of != "step":
            ctx.worker_step_all(loss)
            ctx.aggregate()
        graph.replay()
        check("replayed", B)
        check([1, 0], 2500)
        check(None, B)
