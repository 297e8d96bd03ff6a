"""What is timed on the layer-stack library: the calls that a training program makes, over the sizes it makes them at.

Six kinds of pass, all through the binding of the C ABI:

  step       lga_forward_layered + lga_backward_layered with the fused per-layer Adam: one training step of a stack
  mbmajor    lga_step_mbmajor: the same step in the comparison order, one micro-batch per launch
  forward    lga_forward_layer: one layer over all micro-batches (a device of the modular pipeline runs these)
  backward   lga_backward_layer without Adam: recompute, input gradient and weight gradients of one layer
  attention  lga_op_attention_fwd + lga_op_attention_bwd: the fused attention, forward and backward
  widehead   lga_op_attention_gemm_fwd + _bwd: attention of heads beyond the fused kernels, workspace kept

Weights are N(0, 0.02^2) matrices, gains around 1 and small biases; activations and output gradients N(0, 1) in the
pass's own data type; half precision multiplies the output gradient by a loss scale and tests the gradients, as a
mixed-precision program does.
"""
import math

import numpy as np
import torch

from paper_2106_02679_amd import binding as B

DTYPES = {"fp32": (B.LGA_FP32, torch.float32, 4), "bf16": (B.LGA_BF16, torch.bfloat16, 2), "fp16": (B.LGA_FP16, torch.float16, 2)}
LR, BETA1, BETA2, EPS = 1e-6, 0.9, 0.999, 1e-8
STACK_KINDS = ("step", "mbmajor", "forward", "backward")


def _stack_case(name, kind, dtype, layers, d, heads, ff, s, b, n_micro, group, full=0, host_weights=True, loss_scale=0.0):
    c = dict(kind=kind, dtype=dtype, layers=layers, d=d, heads=heads, ff=ff, s=s, b=b, n_micro=n_micro, group=group,
             full=full, host_weights=host_weights, loss_scale=loss_scale)
    return dict(c, name=name) if name else c


def _attention_case(name, kind, dtype, seqs, s, heads, dh, full=0):
    c = dict(kind=kind, dtype=dtype, seqs=seqs, s=s, heads=heads, dh=dh, full=full)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest workload of the repository, in fp32: a step of short launches, bound by their number
        _stack_case("tiny_fp32_step", "step", "fp32", 2, 64, 4, 256, 32, 2, 4, 4),
        # the smallest 16-bit stack that is run as a smoke test: few workgroups per launch
        _stack_case("small_bf16_step", "step", "bf16", 2, 128, 2, 512, 128, 1, 4, 2),
        # fp32 at the size of the paper's X_16, as its encoder: what a run in full precision waits for
        _stack_case("x16_encoder_fp32_step", "step", "fp32", 2, 256, 8, 1024, 256, 2, 4, 4, full=1),
        # GPT-2 small, one of its twelve layers over the step's 32768 tokens: the two directions of a modular pipeline
        _stack_case("gpt2_small_forward", "forward", "bf16", 1, 768, 12, 3072, 1024, 4, 8, 8),
        _stack_case("gpt2_small_backward", "backward", "bf16", 1, 768, 12, 3072, 1024, 4, 8, 8),
        # the same model in the comparison order: one micro-batch of 4096 tokens per launch
        _stack_case("gpt2_small_mbmajor", "mbmajor", "bf16", 2, 768, 12, 3072, 1024, 4, 2, 1),
        # one layer of the middle configuration (d 2048) with the step's 65536 tokens: the ordinary training step
        _stack_case("mid_step", "step", "bf16", 1, 2048, 16, 8192, 2048, 2, 16, 8),
        # half precision with a loss scale at T-NLG's width: heads of 152 (padded kernels), an odd sequence length
        _stack_case("tnlg_fp16_step", "step", "fp16", 1, 4256, 28, 17024, 1000, 1, 4, 2, loss_scale=256.0),
        # one layer of the paper's X_64 as its encoder (no mask), backward
        _stack_case("x64_encoder_backward", "backward", "bf16", 1, 4096, 32, 16384, 1024, 1, 8, 4, full=1),
        # one layer of the GPT-3 share (d 12288), a quarter of its micro-batches: the largest step
        _stack_case("gpt3_share_step", "step", "bf16", 1, 12288, 96, 49152, 2048, 1, 8, 4, host_weights=False),
        # attention of a long context with a ragged last block, forward and backward
        _attention_case("long_context_attention", "attention", "bf16", 1, 8100, 16, 128),
        # attention of the paper's X_108: heads of 216, beyond the fused kernels
        _attention_case("x108_wide_heads", "widehead", "bf16", 2, 1728, 54, 216),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "forward", "backward", "mbmajor", "attention", "widehead"))
    full = int(rng.random() < 0.25)
    if kind == "attention":
        dh = rng.choice((24, 32, 64, 64, 80, 96, 128, 128, 152, 160))
        s = _log(rng, 60, 6000)
        return _attention_case(None, kind, rng.choice(("bf16", "bf16", "fp16")), rng.randint(1, max(1, min(8, 8000 // s))), s,
                               rng.randint(2, 32), dh, full)
    if kind == "widehead":
        return _attention_case(None, kind, rng.choice(("bf16", "fp16")), rng.randint(1, 2), 8 * _log(rng, 20, 220), rng.randint(2, 40),
                               8 * rng.randint(21, 40), full)
    dtype = rng.choice(("bf16", "bf16", "bf16", "fp16", "fp32"))
    for _ in range(1000):
        n_micro = rng.choice((1, 2, 4, 6, 8))
        group = 1 if kind == "mbmajor" else rng.choice([g for g in (1, 2, 3, 4, 8) if n_micro % g == 0])
        b = rng.choice((1, 2, 4))
        if dtype == "fp32":
            dh, heads, s = rng.choice((10, 16, 32, 64)), rng.randint(1, 8), _log(rng, 16, 400)
            ff = rng.choice((4 * dh * heads, rng.randint(30, 1500)))
        else:
            dh, heads, s = rng.choice((32, 64, 64, 96, 128, 128, 152)), _log(rng, 2, 32), _log(rng, 48, 2048)
            ff = 8 * rng.randint(dh * heads // 4, dh * heads // 2) if rng.random() < 0.3 else 4 * dh * heads
        d, tokens = dh * heads, n_micro * b * s
        layers = rng.choice((1, 2)) if kind in ("step", "mbmajor") else 1
        if dtype != "fp32" and (group * b * s) % 8:
            s = (s + 7) // 8 * 8 - rng.choice((0, 8)) if group * b < 8 else s
        if s < 16 or (dtype != "fp32" and (group * b * s) % 8):
            continue
        work = 8.0 * layers * tokens * (4 * d * d + 2 * d * ff)
        if d > 4096 or work > (2e11 if dtype == "fp32" else 3e13) or work < 1e7:
            continue
        return _stack_case(None, kind, dtype, layers, d, heads, ff, s, b, n_micro, group, full,
                           loss_scale=128.0 if dtype == "fp16" and kind in ("step", "mbmajor") else 0.0)
    raise RuntimeError("no case drawn")


# ---- inputs ---------------------------------------------------------------------------------------------------------
NAMES = ("ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_o", "b_o", "ln2_g", "ln2_b", "w_1", "b_1", "w_2", "b_2")


def _shapes(c):
    d, f = c["d"], c["ff"]
    return ((d,), (d,), (d, 3 * d), (3 * d,), (d, d), (d,), (d,), (d,), (d, f), (f,), (f, d), (d,))


def _weights(c, seed):
    """One flat fp32 vector per layer, in the library's order (on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(2 * seed + 1)
    out = []
    for _ in range(c["layers"]):
        parts = []
        for name, shape in zip(NAMES, _shapes(c)):
            t = torch.randn(math.prod(shape), device="cuda", generator=g) * 0.02
            parts.append(t + 1.0 if name.endswith("_g") else t)
        out.append(torch.cat(parts))
    return out


def _activations(c, seed):
    g = torch.Generator(device="cuda").manual_seed(2 * seed)
    shape = (c["n_micro"], c["b"], c["s"], c["d"])
    dt = DTYPES[c["dtype"]][1]
    x = torch.randn(shape, device="cuda", generator=g).to(dt)
    dy = (torch.randn(shape, device="cuda", generator=g) * (c["loss_scale"] or 1.0)).to(dt)
    return x, dy


def _attention_inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(2 * seed)
    dt, d = DTYPES[c["dtype"]][1], c["heads"] * c["dh"]
    qkv = torch.randn(c["seqs"] * c["s"], 3 * d, device="cuda", generator=g).to(dt)
    dout = torch.randn(c["seqs"] * c["s"], d, device="cuda", generator=g).to(dt)
    return qkv, dout


class _Borrowed:
    """An fp32 vector that the stack owns, for torch to look at; it keeps the stack alive."""

    def __init__(self, stack, ptr, count):
        self.stack = stack
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<f4", "data": (ptr, False), "version": 2}


def _view(stack, ptr, count):
    return torch.as_tensor(_Borrowed(stack, ptr, count), device="cuda")


def prepare(case, seed):
    c = case
    code, dt, _ = DTYPES[c["dtype"]]
    if c["kind"] not in STACK_KINDS:
        qkv, dout = _attention_inputs(c, seed)
        st = dict(case=c, qkv=qkv, dout=dout, out=torch.empty_like(dout), dqkv=torch.empty_like(qkv),
                  lse=torch.empty(c["seqs"], c["heads"], c["s"], device="cuda"),
                  delta=torch.empty(c["seqs"], c["heads"], c["s"], device="cuda"))
        if c["kind"] == "widehead":
            st["ws"] = torch.empty(B.lib.lga_op_attention_gemm_workspace_bytes(c["s"], c["heads"]), device="cuda", dtype=torch.uint8)
        return st
    cfg = B.make_config(c["layers"], c["d"], c["heads"], c["ff"], c["s"], c["b"], c["n_micro"], code, group=c["group"],
                        retain_grads=1, attention=B.LGA_ATTN_FULL if c["full"] else B.LGA_ATTN_CAUSAL)
    weights = torch.cat(_weights(c, seed)).cpu().numpy() if c["host_weights"] else None
    x, dy = _activations(c, seed)
    torch.cuda.synchronize()
    stack = B.Stack(cfg, weights)
    st = dict(case=c, stack=stack, x=x, dy=dy, y=torch.empty_like(x), dx=torch.empty_like(x), step=0, grads=None)
    if c["kind"] in ("step", "mbmajor"):
        st["w"] = [_view(stack, *stack.params(l)) for l in range(c["layers"])]
        st["mv"] = []
        for l in range(c["layers"]):
            m, v, n = stack.moments(l)
            st["mv"] += [_view(stack, m, n), _view(stack, v, n)]
    if c["kind"] == "backward":
        stack.forward_layer(0, x.data_ptr(), st["y"].data_ptr())
    return st


def _grads(st):
    if st["grads"] is None:
        st["grads"] = [_view(st["stack"], *st["stack"].grads(l)) for l in range(st["case"]["layers"])]
    return st["grads"]


def run(state):
    st, c = state, state["case"]
    code = DTYPES[c["dtype"]][0]
    if c["kind"] not in STACK_KINDS:
        qkv, out, lse, dout, dqkv, delta = (st[k].data_ptr() for k in ("qkv", "out", "lse", "dout", "dqkv", "delta"))
        shape = (c["seqs"], c["s"], c["heads"], c["dh"], 0 if c["full"] else 1)
        if c["kind"] == "attention":
            B.check(B.lib.lga_op_attention_fwd(code, 1, qkv, out, lse, *shape, None))
            B.check(B.lib.lga_op_attention_bwd(code, 1, qkv, out, lse, dout, dqkv, delta, *shape, None))
        else:
            ws, n = st["ws"].data_ptr(), st["ws"].numel()
            B.check(B.lib.lga_op_attention_gemm_fwd(code, qkv, out, lse, *shape, ws, n, None))
            B.check(B.lib.lga_op_attention_gemm_bwd(code, qkv, out, lse, dout, dqkv, delta, *shape, ws, n, None))
        return {"out": st["out"], "lse": st["lse"], "dqkv": st["dqkv"]}
    stack, x, dy, y, dx = st["stack"], st["x"].data_ptr(), st["dy"].data_ptr(), st["y"].data_ptr(), st["dx"].data_ptr()
    if c["kind"] == "forward":
        stack.forward_layer(0, x, y)
        return {"y": st["y"]}
    if c["kind"] == "backward":
        stack.backward_layer(0, dy, dx, None)
        return {"dx": st["dx"], "grads": _grads(st)}
    st["step"] += 1
    adam = B.lga_adam(LR, BETA1, BETA2, EPS, st["step"], c["loss_scale"], 1 if c["loss_scale"] else 0)
    if c["kind"] == "step":
        stack.forward_layered(x, y)
        stack.backward_layered(dy, dx, adam)
    else:
        stack.step_mbmajor(x, dy, y, dx, adam)
    return {"y": st["y"], "dx": st["dx"], "grads": _grads(st), "weights": st["w"], "moments": st["mv"]}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def work(case):
    c = case
    e = DTYPES[c["dtype"]][2]
    pairs = 1.0 if c["full"] else 0.5                                   # share of the (query, key) pairs that are visible
    if c["kind"] not in STACK_KINDS:
        d = c["heads"] * c["dh"]
        product = 2.0 * c["seqs"] * c["s"] ** 2 * d * pairs
        act = c["seqs"] * c["s"] * d * e
        return {"bytes": act * (3 + 1 + 1 + 3) + 4.0 * c["seqs"] * c["s"] * c["heads"], "flops": 7 * product}
    d, f = c["d"], c["ff"]
    tokens = c["n_micro"] * c["b"] * c["s"]
    mats, params = 4 * d * d + 2 * d * f, 4 * d * d + 2 * d * f + 9 * d + f
    act = tokens * d * e
    product = 2.0 * tokens * c["s"] * d * pairs                         # one attention product of a layer
    forward = 2.0 * tokens * mats + 2 * product
    # recomputed from the layer's input except for its last product, then two products per matrix and five of attention
    backward = forward - 2.0 * tokens * d * f + 4.0 * tokens * mats + 5 * product
    if c["kind"] == "forward":
        return {"bytes": 2 * act + params * e, "flops": forward}
    if c["kind"] == "backward":
        return {"bytes": 3 * act + params * (e + 4), "flops": backward}
    # weights and moments are read and written, the gradients written
    return {"bytes": 4 * act + c["layers"] * (2 * act + params * (24.0 + 4 + (2 if e == 2 else 0))), "flops": c["layers"] * (forward + backward)}


def tolerance(case):
    """Relative errors of another correct implementation at the same precision."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3}
    half = case["dtype"] == "fp16"
    if case["kind"] not in STACK_KINDS:
        return {"rel": 1.25e-3 if half else 1e-2, "max": 0.05 if half else 0.4}
    return {"rel": 4e-3 if half else 2e-2, "max": 0.16 if half else 0.8}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------
def _heads_attention(q, k, v, full):
    """softmax(q k^T / sqrt(dh)) v over [heads, s, dh]; also the log-sum-exp of the scaled scores."""
    s = q.shape[1]
    scores = q @ k.transpose(1, 2) / math.sqrt(q.shape[2])
    if not full:
        scores = scores.masked_fill(torch.ones(s, s, dtype=torch.bool, device=q.device).triu(1), -math.inf)
    lse = torch.logsumexp(scores, -1)
    return torch.exp(scores - lse[..., None]) @ v, lse


def _exact_attention(c, seed):
    qkv, dout = (t.double() for t in _attention_inputs(c, seed))
    n, s, heads, dh = c["seqs"], c["s"], c["heads"], c["dh"]
    qkv, dout = qkv.view(n, s, 3, heads, dh), dout.view(n, s, heads, dh)
    out, dqkv = torch.empty_like(dout), torch.empty_like(qkv)
    lse = torch.empty(n, heads, s, device="cuda", dtype=torch.float64)
    for i in range(n):
        for h in range(heads):
            part = qkv[i, :, :, h].detach().clone().requires_grad_()
            o, l = _heads_attention(part[None, :, 0], part[None, :, 1], part[None, :, 2], c["full"])
            o.backward(dout[i, :, h][None])
            out[i, :, h], lse[i, h], dqkv[i, :, :, h] = o[0].detach(), l[0].detach(), part.grad
    d = heads * dh
    return {"out": out.view(n * s, d), "lse": lse, "dqkv": dqkv.reshape(n * s, 3 * d)}


def _norm(x, g, b):
    mean = x.mean(-1, keepdim=True)
    var = ((x - mean) ** 2).mean(-1, keepdim=True)
    return (x - mean) / torch.sqrt(var + float(np.float32(1e-5))) * g + b


def _layer(c, x, p):
    """x: [b, s, d] of one micro-batch; p: the layer's tensors by name."""
    b, s, d = x.shape
    heads = c["heads"]
    qkv = (_norm(x, p["ln1_g"], p["ln1_b"]) @ p["w_qkv"] + p["b_qkv"]).view(b, s, 3, heads, d // heads).permute(2, 0, 3, 1, 4)
    a = torch.stack([_heads_attention(qkv[0, i], qkv[1, i], qkv[2, i], c["full"])[0] for i in range(b)])
    x1 = x + a.permute(0, 2, 1, 3).reshape(b, s, d) @ p["w_o"] + p["b_o"]
    u = _norm(x1, p["ln2_g"], p["ln2_b"]) @ p["w_1"] + p["b_1"]
    return x1 + torch.nn.functional.gelu(u, approximate="tanh") @ p["w_2"] + p["b_2"]


def exact(case, seed):
    c = case
    if c["kind"] not in STACK_KINDS:
        return _exact_attention(c, seed)
    if not c["host_weights"]:
        return None
    flats = [w.double().requires_grad_() for w in _weights(c, seed)]
    layers = []
    for flat in flats:
        parts = torch.split(flat, [math.prod(s) for s in _shapes(c)])
        layers.append({n: t.view(s) for n, t, s in zip(NAMES, parts, _shapes(c))})
    x, dy = (t.double() for t in _activations(c, seed))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    for mu in range(c["n_micro"]):
        xin = x[mu].detach().clone().requires_grad_()
        h = xin
        for p in layers:
            h = _layer(c, h, p)
        y[mu] = h.detach()
        if c["kind"] != "forward":
            h.backward(dy[mu], retain_graph=True)
            dx[mu] = xin.grad
        del h
    if c["kind"] == "forward":
        return {"y": y}
    grads = [f.grad for f in flats]
    if c["kind"] == "backward":
        return {"dx": dx, "grads": grads}
    lr, b1, b2, eps = (float(np.float32(v)) for v in (LR, BETA1, BETA2, EPS))
    weights, moments = [], []
    for f, g in zip(flats, grads):
        g = g / (c["loss_scale"] or 1.0)
        m, v = (1 - b1) * g, (1 - b2) * g * g
        weights.append(f.detach() - lr * (m / (1 - b1)) / (torch.sqrt(v / (1 - b2)) + eps))
        moments += [m, v]
    return {"y": y, "dx": dx, "grads": grads, "weights": weights, "moments": moments}
