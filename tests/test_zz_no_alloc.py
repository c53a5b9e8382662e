"""antdt_bind_static, the entry point for callers that cannot allocate: the library's static
device buffer serves as the workspace and every kernel goes to the caller's stream.  Its
results are compared with those of antdt_bind (caller-allocated workspace, library streams) on
the same inputs: integers identical, floating point within the fp32 tolerance (the kernels and
their order of addition are the same, so they are in fact equal bit for bit, which is asserted
too).  Two bindings in a row share the buffer, the second for a smaller model."""
import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu

MID_BF = wl.RankingConfig("mid-bf16gemm", 5, 100_000, 32, "f32", "elementwise", 13, (173, 256, 128, 64, 1), "bf16",
                          20, 1.1, (300, 37, 0, 663), wl.SEED0 + 201)


def _inputs(cfg):
    tables, flat, batch = wl.make_tables(cfg), wl.make_mlp_params(cfg), wl.make_batch(cfg, 0)
    rng = np.random.default_rng(cfg.seed + 999)
    n_rows = cfg.num_fields * cfg.rows_per_field
    shape = (n_rows, cfg.dim) if cfg.adagrad_state == "elementwise" else (n_rows,)
    state = (rng.random(shape, dtype=np.float32) * np.float32(1e-4)).astype(np.float32)
    fstate = (rng.random(flat.shape, dtype=np.float32) * np.float32(1e-4)).astype(np.float32)
    return tables, state, flat, fstate, batch


def _iteration(cfg, inputs, static, mask=None):
    from gpu_helpers import GpuRun
    tables, state, flat, fstate, batch = inputs
    run = GpuRun(cfg, tables, flat, state, fstate, max_batch=batch.batch, max_shards=len(cfg.shard_sizes),
                 max_nnz=int(batch.field_ptr[-1]), static=static)
    run.set_batch(batch)
    run.iteration(cfg.shard_sizes, batched=True, mask=mask)
    return run


def _same(a, b, what):
    a, b = np.asarray(a), np.asarray(b)
    assert a.shape == b.shape, what
    if a.dtype.kind in "iu":
        assert np.array_equal(a, b), what
    else:
        d = np.abs(a.astype(np.float64) - b.astype(np.float64))
        scale = max(float(np.abs(b).max()) if b.size else 0.0, 1e-30)
        assert float(d.max() if d.size else 0.0) <= 1e-5 * scale, what
        assert np.array_equal(a, b), what + " (bitwise)"


def _compare(ref, got):
    _same(got.loss.cpu().numpy(), ref.loss.cpu().numpy(), "shard losses")
    for k, (r, g) in enumerate(zip(ref.shard_out, got.shard_out)):
        for name, x, y in zip(("pooled input", "dense gradient", "d loss / d pooled"), r, g):
            _same(y, x, f"{name}, shard {k}")
    _same(got.g_dense, ref.g_dense, "aggregated dense gradient")
    for f, (r, g) in enumerate(zip(ref.coalesced, got.coalesced)):
        for name, x, y in zip(("unique ids", "segment offsets", "grouping", "coalesced gradient"), r, g):
            _same(y, x, f"{name}, field {f}")
    _same(got.tables.float().cpu().numpy(), ref.tables.float().cpu().numpy(), "updated tables")
    _same(got.state.cpu().numpy(), ref.state.cpu().numpy(), "updated table accumulators")
    _same(got.params.cpu().numpy(), ref.params.cpu().numpy(), "updated MLP parameters")
    _same(got.pstate.cpu().numpy(), ref.pstate.cpu().numpy(), "updated MLP accumulators")


def test_static_binding_matches_the_allocated_workspace_twice_in_a_row():
    import paper_2404_09679_amd as A
    big, small = MID_BF, wl.CONFIGS[1]
    in_big, in_small = _inputs(big), _inputs(small)
    ref_big = _iteration(big, in_big, static=False)
    ref_small = _iteration(small, in_small, static=False, mask=(1, 0, 1, 1))
    torch.cuda.synchronize()
    # first call: a model whose workspace (13 MiB) fills a good part of the static buffer
    got_big = _iteration(big, in_big, static=True)
    _compare(ref_big, got_big)
    assert got_big.ctx.workspace_bytes() > 8 << 20
    # second call, smaller input, on the buffer as the first left it (with a mask: the packed
    # lookups go through the staging parts of the buffer as well)
    got_small = _iteration(small, in_small, static=True, mask=(1, 0, 1, 1))
    _compare(ref_small, got_small)
    # the buffer now belongs to the second context: the first must be bound again
    with pytest.raises(A.AntdtError) as e:
        got_big.ctx.set_batch(got_big.d_ids, got_big.batch.field_ptr, got_big.d_off, got_big.d_dense, got_big.d_labels)
    assert e.value.code == -2
    # and a third call on the first context after binding it again
    got_big.ctx.bind_static(got_big.tables, got_big.state, got_big.params, got_big.pstate)
    got_big.set_batch(in_big[4])
    got_big.iteration(big.shard_sizes, batched=True)
    ref_big.set_batch(in_big[4])
    ref_big.iteration(big.shard_sizes, batched=True)
    _compare(ref_big, got_big)


def test_static_binding_allocates_no_device_memory():
    from gpu_helpers import GpuRun
    cfg = MID_BF
    tables, state, flat, fstate, batch = _inputs(cfg)
    warm = GpuRun(cfg, tables, flat, state, fstate, max_batch=batch.batch, max_shards=len(cfg.shard_sizes),
                  max_nnz=int(batch.field_ptr[-1]))
    warm.set_batch(batch)
    warm.iteration(cfg.shard_sizes, batched=True)          # every kernel has run once, the code is loaded
    run = GpuRun(cfg, tables, flat, state, fstate, max_batch=batch.batch, max_shards=len(cfg.shard_sizes),
                 max_nnz=int(batch.field_ptr[-1]), static=True)   # (first static binding of this process or not)
    run.set_batch(batch)
    loss = torch.zeros(len(cfg.shard_sizes), device="cuda:0")
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    reserved0 = torch.cuda.memory_reserved()
    run.ctx.bind_static(run.tables, run.state, run.params, run.pstate)
    run.ctx.set_batch(run.d_ids, batch.field_ptr, run.d_off, run.d_dense, run.d_labels)
    run.ctx.assign_shard(batch.batch, len(cfg.shard_sizes), sizes=cfg.shard_sizes)
    for _ in range(3):
        run.ctx.worker_step_all(loss)
        run.ctx.aggregate()
        run.ctx.apply_update()
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert torch.cuda.memory_reserved() == reserved0
    # the workspace of this model is 13 MiB: an allocation of it would show
    assert free0 - free1 < (4 << 20), f"device memory shrank by {free0 - free1} bytes"


def test_static_binding_rejects_a_model_beyond_the_buffer():
    import paper_2404_09679_amd as A
    cfg = wl.CONFIGS[2]
    ctx = A.Context(A.model_from_config(cfg))
    assert ctx.workspace_bytes() > 32 << 20
    t = torch.zeros(64, device="cuda:0")
    with pytest.raises(A.AntdtError) as e:
        ctx.bind_static(t, t, t, t)
    assert e.value.code == -3 and str(ctx.workspace_bytes()) in str(e.value) and str(32 << 20) in str(e.value)
