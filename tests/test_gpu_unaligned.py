"""Parameters and gradients at addresses that are not 16-byte aligned (views into one
flat buffer, as an optimizer may keep them): LayerNorm reads them element by element, the
launches that need aligned operands
leave such products to the register-staged or strided GEMMs, run the LayerNorm on its
own after a split product, and form the weight gradients one by one.  The stage against
the fp64 oracle (bf16 2e-2, the bound of every bf16 stage; fp32 3e-5: unit roundoff 6e-8,
root of 4096 terms, 8 chained products)."""
import ctypes

import pytest
import torch

from paper_2102_07988_amd import synth
from stage_harness import PARAM_KEYS, compare, make_inputs, run_oracle

pytestmark = pytest.mark.gpu

TOL = {"fp32": 3e-5, "bf16": 2e-2}
REF = {}  # the oracle's run of each shape
BIASES = ("ln1_g", "ln1_b", "b_qkv", "b_o", "ln2_g", "ln2_b", "b1", "b2")


def _views(tensors, keys, offset):
    """`keys` as views `offset` elements off an aligned address, the rest as they are."""
    out = {}
    for k, v in tensors.items():
        if k not in keys:
            out[k] = v.clone()
            continue
        flat = torch.empty(v.numel() + 16, dtype=v.dtype, device=v.device)
        out[k] = flat[offset:offset + v.numel()].view(v.shape)
        out[k].copy_(v)
        assert out[k].data_ptr() % 16
    return out


@pytest.mark.parametrize("dtype,H,heads,n", [
    ("bf16", 512, 4, 128), ("bf16", 1024, 16, 200), ("bf16", 96, 3, 33), ("fp32", 256, 4, 100),
])
@pytest.mark.parametrize("what", ["biases", "weights", "grads", "all"])
@pytest.mark.parametrize("offset", [1, 4])
def test_views_into_a_flat_buffer(dtype, H, heads, n, what, offset):
    from paper_2102_07988_amd import terapipe as tp
    if dtype == "fp32" and offset == 4:
        offset = 2
    print(f"case {dtype} H={H} heads={heads} n={n} {what} offset={offset}", flush=True)
    NL, L, fwd, bwd = 2, n + 40, [40, n], [n, 40]
    params, x, dy = make_inputs(NL, H, L, dtype, (21, 22, 23), True)
    dev = torch.device("cuda:0")
    pk = {"biases": BIASES, "weights": [k for k in PARAM_KEYS if k not in BIASES],
          "grads": [], "all": PARAM_KEYS}[what]
    st = tp.Stage([_views({k: v.to(dev) for k, v in p.items()}, pk, offset) for p in params],
                  H, heads, L, dtype=dtype, wgrad="deferred")
    if what in ("grads", "all"):
        # the same stage over gradients that are views too
        st.grads = [_views(g, PARAM_KEYS, 1) for g in st.grads]
        P, G = (tp.LayerPtrs * NL)(), (tp.LayerPtrs * NL)()
        for i in range(NL):
            for f, k in zip(tp.PARAM_FIELDS, tp.SYNTH_NAMES):
                setattr(P[i], f, st.params[i][k].data_ptr())
                setattr(G[i], f, st.grads[i][k].data_ptr())
        tp.lib.tp_stage_destroy(st._h)
        st._h = ctypes.c_void_p()
        assert tp.lib.tp_stage_init(ctypes.byref(st.cfg), P, G, st.workspace.data_ptr(),
                                    st.workspace.numel(), st.stream.cuda_stream,
                                    ctypes.byref(st._h)) == tp.TP_OK
    key = (dtype, H)
    if key not in REF:
        REF[key] = run_oracle(params, x, dy, H, heads, L, fwd, bwd)
    y, dx = st.run_sequence(x.to(dev), dy.to(dev), fwd, bwd)
    torch.cuda.synchronize()
    got = {"y": y.float().cpu().numpy(), "dx": dx.float().cpu().numpy(),
           "grads": [{k: v.cpu().numpy() for k, v in g.items()} for g in st.grads]}
    compare(got, REF[key], TOL[dtype], f"{dtype} {what}")
