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


# (samples per shard, hidden widths): tiles of 32 (few blocks), 64, 128 and 256 rows and columns in the forward
# and data-gradient products, tiles of 64 and 128 in the weight gradients; no dimension a multiple of its tile
PRODUCT_SHAPES = [((1,), (8,)), ((20, 13), (40, 8)), ((513, 0, 199), (264, 72)), ((2000, 1301), (1032, 136)),
                  ((5003, 3200), (2056, 1544))]


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


# the reduction works on windows of 256 (or 512) sorted lookups: runs of 1 .. 5 lookups, of 15 .. 17 around the length
# from which they are cut into pieces, runs that end at, start at and cross window boundaries or span several
# windows, and a field that ends in the middle of one; the block-per-field sort at 2048 lookups more or fewer
RUN_LENGTHS = [1, 1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 100, 28, 1, 255, 256, 257, 1, 1, 700, 2, 16, 16, 500, 17, 1, 1, 1200, 3]


@pytest.mark.parametrize("dim,table,state,more", [(4, "f32", "elementwise", 0), (32, "f32", "elementwise", 3), (256, "f32", "rowwise", 1),
                                                  (8, "bf16", "rowwise", 255), (64, "bf16", "elementwise", 256)])
def test_runs_and_windows(dim, table, state, more, monkeypatch):
    lengths = RUN_LENGTHS + [1] * more
    bag = 5
    total = sum(lengths)
    B = -(-total // bag)
    cfg = _config(f"windows-{dim}", 600 + dim, num_fields=2, rows_per_field=1200, dim=dim, table_dtype=table, adagrad_state=state,
                  layer_sizes=(8,), gemm_dtype="f32", shard_sizes=(B // 3, B - B // 3), max_bag=bag)
    real = wl.make_batch

    def planted(c, index=0):
        b = real(c, index)
        rng = np.random.default_rng(7 + dim)
        ids, offsets, ptr = [], np.zeros((2, B + 1), np.int32), [0]
        for f in range(2):
            rows = rng.permutation(c.rows_per_field)[:len(lengths)]
            field = np.repeat(rows, lengths)
            ids.append(rng.permutation(field).astype(np.int32))
            offsets[f] = np.minimum(np.arange(B + 1) * bag, total)
            ptr.append(ptr[-1] + total)
        return dataclasses.replace(b, ids=np.concatenate(ids), offsets=offsets, field_ptr=np.array(ptr, np.int64))

    monkeypatch.setattr(wl, "make_batch", planted)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)


# enough samples per shard that the weight gradients are formed piece by piece: unequal weights (a piece per shard, the
# longest first) and equal ones (one range cut into pieces), against the update that walks all samples (a per-shard
# view in between keeps it to that)
@pytest.mark.parametrize("sizes", [(1500, 2700, 1100, 3700), (2300,) * 4])
def test_weight_gradient_pieces(sizes):
    import torch
    from gpu_helpers import GpuRun
    from test_gpu_parity import assert_close, make_inputs
    cfg = _config(f"pieces-{sizes[0]}", 700 + sizes[0], num_fields=3, layer_sizes=(1288, 1032), shard_sizes=sizes)
    tables, state, flat, fstate, batch = make_inputs(cfg, nonzero_state=True)
    got = []
    for view in (False, True):
        run = GpuRun(cfg, tables, flat, state, fstate)
        run.set_batch(batch)
        run.ctx.assign_shard(batch.batch, len(sizes), sizes=sizes)
        run.ctx.worker_step_all(torch.zeros(len(sizes), device="cuda:0"))
        if view:
            run.ctx.view_shard_grads(0)
        run.ctx.aggregate()
        run.ctx.apply_update()
        run.ctx.worker_step_all(torch.zeros(len(sizes), device="cuda:0"))   # (from the updated bf16 copies)
        torch.cuda.synchronize()
        got.append((run.params.cpu().numpy().copy(), run.pstate.cpu().numpy().copy(), run.ctx.view_pooled(0).float().cpu().numpy().copy(),
                    run.ctx.view_shard_grads(1)[1].cpu().numpy().copy()))
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
    real = wl.make_batch

    def planted(c, index=0):
        b = real(c, index)
        rng = np.random.default_rng(11 + rows)
        offsets = np.zeros((F, B + 1), np.int32)
        for f, n in enumerate(sizes):
            offsets[f, 1:] = np.sort(rng.integers(0, n + 1, B))
            offsets[f, -1] = n
        ids = rng.integers(0, rows, sum(sizes)).astype(np.int32)
        return dataclasses.replace(b, ids=ids, offsets=offsets, field_ptr=np.cumsum([0] + sizes).astype(np.int64))

    monkeypatch.setattr(wl, "make_batch", planted)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, batched=True, nonzero_state=True)
    check_iteration(cfg, cfg.shard_sizes, tol=TOL32, mask=(1, 1, 0, 1), nonzero_state=True)


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
