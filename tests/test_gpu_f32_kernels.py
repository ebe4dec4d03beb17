"""fp32 matrix-core kernels (the GEMM of fp32 stages; the attention of fp32 stages
and of bf16 stages with heads of 16 or 32) at the edges of their tiles: slices of 1
row and of one more and one less than a tile, prefixes of more than one tile per
wave (8 waves x 32 keys), split reductions, the 128 x 128 tiles of products with at
least 256 of them.

Tolerances (rel-L2 against the fp64 oracle): fp32 3e-5, the fp32 unit roundoff
6e-8 times the root of the longest reduction (4096) times the 8 products chained
from input to gradient; bf16 2e-2, the bound of every bf16 stage."""
import pytest

from stage_harness import (PARAM_KEYS, compare, make_batch_inputs, make_inputs, run_gpu,
                           run_gpu_batch, run_oracle, run_oracle_batch)

pytestmark = pytest.mark.gpu

TOL = {"fp32": 3e-5, "bf16": 2e-2}


@pytest.mark.parametrize("dtype,H,heads,L,fwd,bwd,wgrad", [
    ("fp32", 128, 1, 301, [33, 1, 255, 12], [31, 270], "per_slice"),    # d = 128, 4 waves
    ("fp32", 192, 3, 321, [64, 257], [1, 63, 257], "deferred"),         # d = 64
    ("fp32", 48, 3, 290, [289, 1], [145, 145], "per_slice"),            # d = 16
    ("fp32", 1024, 8, 40, [40], [7, 33], "deferred"),                   # 128 x 128 dW tiles
    ("bf16", 96, 3, 600, [31, 33, 300, 236], [300, 300], "deferred"),   # d = 32
    ("bf16", 48, 3, 290, [289, 1], [1, 289], "per_slice"),              # d = 16
])
def test_edges(dtype, H, heads, L, fwd, bwd, wgrad):
    print(f"case {dtype} H={H} heads={heads} L={L} fwd={fwd} bwd={bwd} {wgrad}", flush=True)
    params, x, dy = make_inputs(1, H, L, dtype, (51, 52, 53), True)
    got = run_gpu(params, x, dy, H, heads, L, dtype, fwd, bwd, wgrad)
    ref = run_oracle(params, x, dy, H, heads, L, fwd, bwd)
    compare(got, ref, TOL[dtype], f"{dtype} d={H // heads}")
    # every sum has a fixed order: a second run gives the same bits
    again = run_gpu(params, x, dy, H, heads, L, dtype, fwd, bwd, wgrad)
    assert (got["dx"] == again["dx"]).all()
    assert all((got["grads"][0][k] == again["grads"][0][k]).all() for k in PARAM_KEYS)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_batch_slices(dtype):
    H, heads, L = 96, 3, 75
    print(f"case batch {dtype} H={H} heads={heads} L={L} b=3", flush=True)
    params, x, dy = make_batch_inputs(1, H, L, 3, dtype, (54, 55, 56), True)
    got = run_gpu_batch(params, x, dy, H, heads, L, dtype, [40, 35], [8, 67])
    ref = run_oracle_batch(params, x, dy, H, heads, L, [40, 35], [8, 67])
    compare(got, ref, TOL[dtype], f"batch {dtype}")
