"""Bias and LayerNorm-parameter gradients (the column sums of a layer, one launch):
row counts around the least rows of a chunk (256) and of two (512) and column counts off the 64-column
blocks, stored and added, against the oracle.

Tolerances: fp32 3e-5 (unit roundoff 6e-8, root of 4096 terms, 8 chained products),
bf16 2e-2 (the bound of every bf16 stage)."""
import pytest
import torch

from stage_harness import PARAM_KEYS, compare, make_inputs, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,heads,L", [
    ("bf16", 512, 4, 255), ("bf16", 512, 4, 257), ("bf16", 512, 4, 511), ("bf16", 512, 4, 513),
    ("bf16", 48, 3, 600), ("fp32", 80, 5, 257), ("fp32", 256, 4, 1),
])
@pytest.mark.parametrize("wgrad", ["deferred", "per_slice"])
def test_stored_then_added(dtype, H, heads, L, wgrad):
    from paper_2102_07988_amd import terapipe as tp
    print(f"case {dtype} H={H} heads={heads} L={L} {wgrad}", flush=True)
    params, x, dy = make_inputs(1, H, L, dtype, (71, 72, 73), True)
    dev = torch.device("cuda:0")
    st = tp.Stage([{k: v.to(dev) for k, v in p.items()} for p in params], H, heads, L,
                  dtype=dtype, wgrad=wgrad)
    for v in st.grads[0].values():
        v.fill_(float("nan"))
    y, dx = st.run_sequence(x.to(dev), dy.to(dev), [L], overwrite_grads=True)
    torch.cuda.synchronize()
    first = {k: v.clone() for k, v in st.grads[0].items()}
    got = {"y": y.float().cpu().numpy(), "dx": dx.float().cpu().numpy(),
           "grads": [{k: v.cpu().numpy() for k, v in first.items()}]}
    ref = run_oracle(params, x, dy, H, heads, L, [L])
    compare(got, ref, {"fp32": 3e-5, "bf16": 2e-2}[dtype], f"{dtype} H={H} L={L}")
    st.run_sequence(x.to(dev), dy.to(dev), [L])  # adds the same values once more
    torch.cuda.synchronize()
    for k in PARAM_KEYS:
        a, b = st.grads[0][k], first[k]
        # two identical fp32 sums: exactly twice the first (a split product's last
        # addition rounds once)
        assert torch.allclose(a, 2 * b, rtol=1e-6, atol=0), k
