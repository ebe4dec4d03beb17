"""Byte counts of the kernel classes: whichever LayerNorms run in a product's split
reduction, the classes' sum is the stage's algorithmic traffic (a LayerNorm of its own
reads the product's output rows once more)."""
import pytest
import torch

from paper_2102_07988_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,heads,n", [(512, 4, 128), (1024, 16, 200), (512, 16, 64)])
def test_bytes_of_one_slice(H, heads, n):
    from paper_2102_07988_amd import terapipe as tp
    NL, e, A, F = 2, 2, H, 4 * H
    print(f"case H={H} heads={heads} n={n}", flush=True)
    dev = torch.device("cuda:0")
    params = synth.stage_params(NL, H, seed=1, dtype=torch.bfloat16, device=dev)
    x = synth.hidden_states(n, H, seed=2, dtype=torch.bfloat16, device=dev)
    dy = synth.upstream_grad(n, H, seed=3, dtype=torch.bfloat16, device=dev)
    st = tp.Stage(params, H, heads, n, dtype="bf16", wgrad="deferred")
    st.reset(overwrite_grads=True)
    st.enable_kernel_timing(True)
    st.forward(0, n, x)
    fwd = st.kernel_stats()
    st.backward(0, n, dy)
    bwd = st.kernel_stats()
    row, weights = n * H * e, (4 * A * H + 2 * F * H) * e
    own = fwd["layernorm"]["launches"]
    products = weights + e * n * ((H + 3 * A) + (A + 2 * H) + (H + 2 * F) + (F + 2 * H))
    attn = 4 * n * A * e
    total = NL * (products + attn) + (2 * own + (2 * NL - own)) * row
    assert sum(s["bytes"] for s in fwd.values()) == pytest.approx(total, rel=1e-12)
    own = bwd["layernorm"]["launches"] if "layernorm" in bwd else 0
    products = weights + e * n * ((H + 2 * F) + (F + H) + (H + A) + (3 * A + H))
    attn = 8 * n * A * e  # q, dO, dq, o, K, V rows; dK and dV rows of the slice's own keys
    dw = e * n * ((H + F) * 2 + (H + A) + (3 * A + H)) + 2 * weights
    resid = 4 if H // heads >= 64 else e  # the residual stream of the mixed-precision path
    sums = n * ((4 * H + F + 3 * A) * e + 2 * H * resid)
    total = NL * (products + attn + dw + sums) + (4 * own + 3 * (2 * NL - own)) * row
    assert sum(s["bytes"] for s in bwd.values()) == pytest.approx(total, rel=1e-12)
