"""GPU parity of kernel variants at the sizes where their tiling can go wrong: one sample more or
fewer than a tile, remainders in every dimension, the smallest and largest problem a variant is
chosen for.  Same oracle and tolerances as test_gpu_parity.py."""
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
