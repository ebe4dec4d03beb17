"""bf16 LDS-DMA GEMM at the edges of its tiles: slices of any number of rows (1, one
under and over a tile), weight-gradient reductions over any number of tokens (the
last k-tile of 1 to 63 tokens is cleared in LDS), and widths that are not whole
k-tiles (heads of 16 and 32).  The stage against the fp64 oracle; rel-L2 2e-2, the
bound of every bf16 stage (observed 2e-3 to 5e-3)."""
import pytest

from stage_harness import (compare, make_batch_inputs, make_inputs, run_gpu, run_gpu_batch,
                           run_oracle, run_oracle_batch)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,heads,L,fwd,bwd,wgrad", [
    (512, 4, 333, [1, 131, 63, 138], [65, 129, 139], "per_slice"),
    (512, 4, 333, [1, 131, 63, 138], [333], "deferred"),         # 333 = 5 * 64 + 13 tokens
    (640, 5, 257, [257], [255, 2], "per_slice"),                 # 2-token reduction
    (1024, 8, 97, [33, 31, 33], [97], "deferred"),
    (432, 27, 71, [7, 64], [71], "deferred"),                    # K = 432, 1296, 1728
    (96, 3, 130, [129, 1], [1, 129], "per_slice"),               # K = 96, 288, 384
])
def test_edges(H, heads, L, fwd, bwd, wgrad):
    print(f"case H={H} heads={heads} L={L} fwd={fwd} bwd={bwd} {wgrad}", flush=True)
    params, x, dy = make_inputs(1, H, L, "bf16", (61, 62, 63), True)
    got = run_gpu(params, x, dy, H, heads, L, "bf16", fwd, bwd, wgrad, overwrite_grads=True)
    ref = run_oracle(params, x, dy, H, heads, L, fwd, bwd)
    compare(got, ref, 2e-2, f"H={H} {wgrad}")


def test_ragged_batch():
    H, heads, L = 384, 3, 77
    print(f"case batch H={H} heads={heads} L={L} b=3", flush=True)
    params, x, dy = make_batch_inputs(1, H, L, 3, "bf16", (64, 65, 66), True)
    got = run_gpu_batch(params, x, dy, H, heads, L, "bf16", [13, 64], [40, 37], "deferred")
    ref = run_oracle_batch(params, x, dy, H, heads, L, [13, 64], [40, 37])
    compare(got, ref, 2e-2, "ragged batch")
