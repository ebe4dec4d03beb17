"""The attention backward's key / value gradient rows over backward slices longer
than the stored-dS chunk (1024 query rows): the sequence's first slice stores rows
that later chunks and slices add to, a slice's own keys leave as bf16 rows of its
last chunk, with slice edges inside a 32-key block, and the streaming dQ kernel runs
split and unsplit.  The workspace holds NaN before the sequence: nothing may read a
row that was not written.  Whole-sequence float64 reference; rel-L2 2e-2, the bound
of every bf16 stage."""
import pytest
import torch

from oracle.full import stage_forward_backward
from paper_2102_07988_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,heads,L,bwd", [
    (1024, 16, 1500, [299, 1201]),      # d = 64: chunks of 1024 and 177 rows
    (1024, 8, 2100, [699, 1401]),       # d = 128: the second slice adds in two chunks
    (1024, 8, 2100, [1, 2098, 1]),      # one-row slices at both ends
])
def test_rows_of_long_backward_slices(H, heads, L, bwd):
    from paper_2102_07988_amd import terapipe as tp
    print(f"case H={H} heads={heads} L={L} bwd={bwd}", flush=True)
    dev = torch.device("cuda:0")
    params = synth.stage_params(1, H, seed=81, dtype=torch.bfloat16, randomize_ln=True)
    x = synth.hidden_states(L, H, seed=82, dtype=torch.bfloat16)
    dy = synth.upstream_grad(L, H, seed=83, dtype=torch.bfloat16)
    st = tp.Stage([{k: v.to(dev) for k, v in p.items()} for p in params], H, heads, L,
                  dtype="bf16", wgrad="deferred")
    st.workspace.fill_(255)  # NaN in every format
    y, dx = st.run_sequence(x.to(dev), dy.to(dev), [L], bwd, overwrite_grads=True)
    torch.cuda.synchronize()
    ry, rdx, rg = stage_forward_backward(params, x, dy, heads)
    got = dict({"y": y, "dx": dx}, **st.grads[0])
    ref = dict({"y": ry, "dx": rdx}, **rg[0])
    errs = {k: float((got[k].double().cpu() - ref[k].double()).norm() / ref[k].double().norm())
            for k in ref}
    print(errs, flush=True)
    assert all(v <= 2e-2 for v in errs.values()), errs
