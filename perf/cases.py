"""Performance cases of the stage engine: what a training program has one pipeline stage do.

A case is one training iteration of a stage (or, where `direction` says so, the
forward pass alone) through the binding: start a sequence, run the forward of
every token slice in order, then the backward of every slice in reverse.  It is
described by

  hidden, heads   residual width and head count (head width hidden / heads)
  layers          Transformer layers in the stage
  seq, slices     sequence length and its token slicing ("256x8" or "100,28,192")
  dtype           "bf16" or "fp32", the stage's data type
  wgrad           "deferred" (weight gradients once a sequence) or "per_slice"
  batch           sequences that move through the stage together
  parts           the stage is one device's shard of this many
  sequences       sequences of one iteration: the first stores its gradients,
                  later ones add to them
  direction       "train" (forward and backward), "forward", or "static" (the
                  forward entry point that allocates nothing)
"""
import math

import torch

from paper_2102_07988_amd import synth
from paper_2102_07988_amd import terapipe as tp

_DEFAULTS = {"layers": 1, "dtype": "bf16", "wgrad": "deferred", "batch": 1, "parts": 1,
             "sequences": 1, "direction": "train"}


def _case(**kw):
    return dict(_DEFAULTS, **kw)


def listed():
    return [
        # one layer of the 175B shape on the benchmark's slicing: the flagship step
        _case(name="wide_12288", hidden=12288, heads=96, seq=2048, slices="256x8"),
        # one device's work when each 175B layer is split over 8 devices: narrow
        # products on the full residual width
        _case(name="shard8_12288", hidden=12288, heads=96, layers=2, seq=2048, slices="256x8",
              parts=8),
        # the 13B width on a slicing as the planner returns it (long slices first)
        _case(name="planned_5120", hidden=5120, heads=40, seq=2048,
              slices="400,352,304,256,224,176,144,112,80"),
        # the 1.3B stage on the benchmark's slicing
        _case(name="stage_2048", hidden=2048, heads=16, layers=2, seq=2048, slices="256x8"),
        # long context: attention over prefixes of up to 8k tokens
        _case(name="long_2048", hidden=2048, heads=16, seq=8192, slices="512x16"),
        # joint batch and token slicing: 4 sequences in one batch slice
        _case(name="batch4_2048", hidden=2048, heads=16, batch=4, seq=2048,
              slices="512,512,448,352,224"),
        # two sequences an iteration, weight gradients formed slice by slice,
        # head width 64
        _case(name="per_slice_1024", hidden=1024, heads=16, seq=1024, slices="256x4",
              wgrad="per_slice", sequences=2),
        # document lengths and a slicing on no grid at all
        _case(name="ragged_2048", hidden=2048, heads=16, seq=1999,
              slices="301,287,263,251,239,229,223,206"),
        # the finest slices a planner considers, forward only, as a caller that
        # may not allocate runs them
        _case(name="short_fwd_2048", hidden=2048, heads=16, layers=2, seq=256, slices="16x16",
              direction="static"),
        # full-precision stage
        _case(name="fp32_1024", hidden=1024, heads=16, seq=1024, slices="256x4", dtype="fp32"),
        # narrow heads (width 32)
        _case(name="narrow_512", hidden=512, heads=16, layers=2, seq=1024, slices="256x4"),
        # the smallest configuration: launches and host work
        _case(name="tiny_64", hidden=64, heads=4, seq=32, slices="8,8,16", wgrad="per_slice"),
    ]


def _lens(case):
    s = case["slices"]
    if "x" in s:
        n, k = s.split("x")
        return [int(n)] * int(k)
    return [int(v) for v in s.split(",")]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _slicing(rng, seq, most):
    """A slicing of seq tokens: equal slices, or a composition on a grid of 1, 8 or 16 tokens."""
    k = max(1, min(seq, round(_log_uniform(rng, 1, most))))
    if rng.random() < 0.4:
        n = -(-seq // k)
        lens = [n] * (seq // n) + ([seq % n] if seq % n else [])
        return ",".join(str(v) for v in lens)
    grid = rng.choice((1, 8, 16))
    units = max(1, seq // grid)
    k = min(k, units)
    cuts = sorted(rng.sample(range(1, units), k - 1)) if k > 1 else []
    edges = [0] + [c * grid for c in cuts] + [seq]
    return ",".join(str(b - a) for a, b in zip(edges, edges[1:]))


def draw(rng):
    """One more case of the ranges above: mostly bf16 stages of head width 64 or
    128, hidden sizes 256 to 5120 (12288 as a shard) and up to 4096 tokens; some
    narrow-headed bf16 and fp32 stages up to 2048 wide and 1024 tokens long."""
    while True:
        kind = rng.random()
        if kind < 0.75:
            d = rng.choice((64, 128, 128))
            heads = max(1, round(_log_uniform(rng, 256, 5120) / d))
            seq = round(_log_uniform(rng, 64, 4096))
            dtype, most = "bf16", 16
        else:
            dtype = "bf16" if kind < 0.88 else "fp32"
            d = rng.choice((16, 32)) if dtype == "bf16" else rng.choice((32, 64, 128))
            heads = max(1, round(_log_uniform(rng, 64, 2048) / d))
            seq = round(_log_uniform(rng, 32, 1024))
            most = 8
        parts = 1
        if dtype == "bf16" and d == 128 and rng.random() < 0.15:
            parts = rng.choice((2, 4, 8))
            heads = 96 if rng.random() < 0.3 and parts >= 4 else -(-heads // parts) * parts
        direction = rng.choice(("train", "train", "train", "forward"))
        case = _case(hidden=heads * d, heads=heads, layers=rng.choice((1, 1, 2)), seq=seq,
                     slices=_slicing(rng, seq, most), dtype=dtype,
                     wgrad=rng.choice(("deferred", "deferred", "per_slice")),
                     batch=rng.choice((1, 1, 1, 2, 4)), parts=parts,
                     sequences=rng.choice((1, 1, 2)), direction=direction)
        if direction != "train":
            case["sequences"] = 1
        limit = 1.5e13 if dtype == "bf16" and d >= 64 else 4e11
        if work(case)["flops"] <= limit:
            return case


def _inputs(case, seed):
    dev = torch.device("cuda:0")
    dt = tp.torch_dtype(case["dtype"])
    H, L, b = case["hidden"], case["seq"], case["batch"]
    params = synth.stage_params(case["layers"], H, seed=3 * seed + 1, dtype=dt, device=dev,
                                randomize_ln=True, op_parts=case["parts"])
    shape = (L, H) if b == 1 else (L, b, H)
    xs = [synth.normal(shape, 3 * seed, 1 + 10 * i, dtype=dt, device=dev)
          for i in range(case["sequences"])]
    dys = [synth.normal(shape, 3 * seed + 2, 2 + 10 * i, dtype=dt, device=dev)
           for i in range(case["sequences"])]
    return params, xs, dys


def prepare(case, seed):
    params, xs, dys = _inputs(case, seed)
    stage = tp.Stage(params, case["hidden"], case["heads"], case["seq"], dtype=case["dtype"],
                     wgrad=case["wgrad"], batch=case["batch"], op_parts=case["parts"])
    bounds, pos = [], 0
    for n in _lens(case):
        bounds.append((pos, pos + n))
        pos += n
    assert pos == case["seq"]
    return {"stage": stage, "x": xs, "dy": dys, "y": [torch.empty_like(x) for x in xs],
            "dx": [torch.empty_like(v) for v in dys], "bounds": bounds,
            "direction": case["direction"]}


def run(state):
    st, bounds, train = state["stage"], state["bounds"], state["direction"] == "train"
    fwd = st.forward_static if state["direction"] == "static" else st.forward
    for i, (x, y, dy, dx) in enumerate(zip(state["x"], state["y"], state["dy"], state["dx"])):
        st.reset(overwrite_grads=train and i == 0, reuse_wqkv_copy=i > 0)
        for l, r in bounds:
            fwd(l, r, x[l:r], out=y[l:r])
        if train:
            for l, r in reversed(bounds):
                st.backward(l, r, dy[l:r], out=dx[l:r])
    if not train:
        return {"y": state["y"]}
    return {"y": state["y"], "dx": state["dx"], "grads": st.grads}


def work(case):
    """Least bytes (parameters, inputs and outputs once each) and flops (the four
    projections, and 4 A flops a causal (query, key) pair; backward twice that)."""
    H, L, p = case["hidden"], case["seq"], case["parts"]
    A, F = H // p, 4 * H // p
    e = 4 if case["dtype"] == "fp32" else 2
    n = L * case["batch"] * case["sequences"]
    weights = 4 * A * H + 2 * F * H + 3 * A + F + 6 * H
    pairs = L * (L + 1) // 2 * case["batch"] * case["sequences"]
    fwd = 2.0 * n * (4 * A * H + 2 * F * H) + 4.0 * A * pairs
    train = case["direction"] == "train"
    nbytes = case["layers"] * weights * (e + (4 if train else 0)) + n * H * e * (4 if train else 2)
    return {"bytes": float(nbytes), "flops": case["layers"] * fwd * (3 if train else 1)}


def tolerance(case):
    """About four times the error against float64 measured over the ranges: 1.3e-6
    for fp32, 5e-3 for bf16 and 1.3e-2 for bf16 at the widest residual stream,
    whose softmax rows are sharp and amplify the rounding of q and k."""
    if case["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 2e-4}
    return {"rel": 0.03 if case["hidden"] > 8192 else 0.02, "max": 0.5}


def exact(case, seed):
    """The same iteration over whole sequences in float64, by autograd."""
    H, L, b, p = case["hidden"], case["seq"], case["batch"], case["parts"]
    heads, d = case["heads"] // p, H // case["heads"]
    A = heads * d
    if work(case)["flops"] > 4e13 or b * heads * L * L > 2.5e9:
        return None
    params, xs, dys = _inputs(case, seed)
    train = case["direction"] == "train"
    params = [{k: v.double().requires_grad_(train) for k, v in q.items()} for q in params]
    mask = torch.ones(L, L, dtype=torch.bool, device="cuda:0").triu(1)
    lin, norm = torch.nn.functional.linear, torch.nn.functional.layer_norm
    ys, dxs = [], []
    for x0, dy0 in zip(xs, dys):
        x0 = x0.double().reshape(L, b, H).requires_grad_(train)
        x = x0
        for q in params:
            u = norm(x, (H,), q["ln1_g"], q["ln1_b"], 1e-5)
            qkv = lin(u, q["w_qkv"], q["b_qkv"]).reshape(L, b, 3, heads, d)
            qh, kh, vh = (t.contiguous() for t in qkv.permute(2, 1, 3, 0, 4))
            s = torch.matmul(qh, kh.transpose(-1, -2).contiguous()) / math.sqrt(d)
            o = torch.matmul(torch.softmax(s.masked_fill(mask, -math.inf), -1), vh)
            del s
            x = x + lin(o.permute(2, 0, 1, 3).reshape(L, b, A), q["w_o"], q["b_o"])
            u = norm(x, (H,), q["ln2_g"], q["ln2_b"], 1e-5)
            z = torch.nn.functional.gelu(lin(u, q["w1"], q["b1"]), approximate="tanh")
            x = x + lin(z, q["w2"], q["b2"])
        shape = dy0.shape
        if train:
            x.backward(dy0.double().reshape(L, b, H))
            dxs.append(x0.grad.reshape(shape))
        ys.append(x.detach().reshape(shape))
    if not train:
        return {"y": ys}
    return {"y": ys, "dx": dxs, "grads": [{k: v.grad for k, v in q.items()} for q in params]}
