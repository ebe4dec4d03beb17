"""An infinite or NaN token stays causal in the fp32 matrix-core attention (fp32
stages, bf16 stages with heads of 16 or 32): a key's weight is 0 for the queries
before it, and such a pair adds nothing whatever the key's value is.  Outputs of
earlier tokens, and input gradients of tokens after one whose upstream gradient is not
finite, have the bits of the run without it; the token itself is not finite."""
import pytest
import torch

from stage_harness import make_batch_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype,H,heads", [
    ("fp32", 48, 3), ("fp32", 96, 3), ("fp32", 128, 2), ("fp32", 256, 2),
    ("bf16", 48, 3), ("bf16", 96, 3),
])
def test_other_tokens_keep_their_bits(dtype, H, heads, value):
    from paper_2102_07988_amd import terapipe as tp
    L, b, fwd, bwd = 75, 2, [40, 35], [8, 67]
    print(f"case {dtype} H={H} heads={heads} L={L} b={b} value={value}", flush=True)
    dev = torch.device("cuda:0")
    params, x, dy = make_batch_inputs(1, H, L, b, dtype, (91, 92, 93), True)
    params = [{k: v.to(dev) for k, v in p.items()} for p in params]
    x, dy = x.to(dev), dy.to(dev)

    def run(x, dy):
        st = tp.Stage(params, H, heads, L, dtype=dtype, wgrad="deferred", batch=b)
        y, dx = st.run_sequence(x, dy, fwd, bwd)
        torch.cuda.synchronize()
        return y, dx

    y0, dx0 = run(x, dy)
    assert torch.isfinite(y0).all() and torch.isfinite(dx0).all()
    # in the middle and at the end of a 32-key tile of each slice
    for t in (17, 31, 51, 74):
        x1 = x.clone()
        x1[t, 0] = value
        y, _ = run(x1, dy)
        assert torch.equal(y[:t], y0[:t]), t
        assert torch.equal(y[:, 1], y0[:, 1]), t  # the other sequence of the batch
        assert not torch.isfinite(y[t, 0]).any(), t
    for t in (0, 33, 67, 74):
        dy1 = dy.clone()
        dy1[t, 0, 0] = value
        _, dx = run(x, dy1)
        assert torch.equal(dx[t + 1:], dx0[t + 1:]), t
        assert torch.equal(dx[:, 1], dx0[:, 1]), t
        assert not torch.isfinite(dx[t, 0]).any(), t
