"""The work that a program built on this library has it do, as cases to be timed.

A program describes a subgraph of memory-intensive ops, plans it once, keeps the plan, the workspace and its buffers,
binds them, and then issues the bound call once per step: `prepare` does the first, `run` the last.

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs (made from the seed alone), plan and bound call
  run(state)           one pass; returns the outputs
  work(case)           bytes and operations that a pass cannot do without
  tolerance(case)      how far another correct implementation of the same precision may be from this one
  exact(case, seed)    what `run` returns, computed by plain torch in float64
"""
from __future__ import annotations

import math

import torch

import workloads as W
from paper_2009_10924_amd import binding as B

DEVICE = "cuda"
DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # a small row softmax on its own: nothing but the latency of one call (the smallest benchmark configuration)
        {"name": "softmax_small", "kind": "softmax", "rows": 64, "cols": 128, "dtype": "f32"},
        # many tiny independent subgraphs in one packed launch: 8 softmaxes, 8 add + bias + LayerNorms, 8 softmax backwards,
        # 4 RMS norms and 4 bias + GELUs (the packed benchmark workload)
        {"name": "pack_small", "kind": "pack", "each": 8, "rows": 64, "cols": 128},
        # scaled and masked attention probabilities of a padded batch (benchmark configuration)
        {"name": "scores", "kind": "scores", "batch": 32, "heads": 12, "q_len": 128, "k_len": 128, "dtype": "f16"},
        # the same for a batch that was cut to its longest sequence, an odd number of keys
        {"name": "scores_ragged", "kind": "scores", "batch": 16, "heads": 12, "q_len": 197, "k_len": 197, "dtype": "f16"},
        # residual + bias + LayerNorm of a forward pass, float32 in and bfloat16 out (benchmark configuration)
        {"name": "layernorm", "kind": "layernorm", "rows": 8192, "cols": 768, "dtype": "f32", "out": "bf16"},
        # its backward: dx and the two column sums dgamma, dbeta (benchmark pattern)
        {"name": "layernorm_backward", "kind": "layernorm_backward", "rows": 8192, "cols": 768, "dtype": "f32"},
        # bias + GELU with the bias gradient of a feed-forward layer (benchmark's headline configuration)
        {"name": "gelu_dbias", "kind": "gelu_dbias", "rows": 16384, "cols": 3072, "dtype": "bf16"},
        # head split + per-head scale + L2 normalisation (benchmark configuration)
        {"name": "transpose_chain", "kind": "transpose_chain", "batch": 64, "seq": 512, "heads": 12, "dim": 64, "dtype": "f32"},
        # tokens x channels to channels x tokens with an odd number of tokens
        {"name": "transpose_ragged", "kind": "transpose", "d0": 64, "d1": 197, "d2": 768, "d3": 1, "perm": "021", "dtype": "bf16"},
        # log-probabilities over a vocabulary, what a cross-entropy reads (the benchmark's largest workload)
        {"name": "vocabulary", "kind": "log_softmax", "rows": 4096, "cols": 128256, "dtype": "bf16"},
        # the same over a vocabulary of odd size, whose rows start at any element
        {"name": "vocabulary_odd", "kind": "log_softmax", "rows": 2048, "cols": 50257, "dtype": "bf16"},
        # the whole backward pass through a transformer block, explored and run as one program (benchmark workload)
        {"name": "block_backward", "kind": "block_backward", "batch": 32, "seq": 128, "heads": 12, "dim": 64, "ffn": 3072, "dtype": "bf16"},
    ]


# ---- more cases of the same ranges -----------------------------------------------------------------------------------
def _log(rng, lo, hi, step=1):
    """An integer of [lo, hi], uniform over its logarithm, a multiple of `step`."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, max(step, v // step * step)))


def _rows(rng, cols, hi, most):
    """Rows for rows of `cols` elements, at most `most` elements in all."""
    return _log(rng, 16, max(17, min(hi, most // cols)))


def draw(rng):
    kind = rng.choice(("softmax", "pack", "scores", "layernorm", "layernorm_backward", "rmsnorm", "rmsnorm_backward", "gelu_dbias",
                       "transpose_chain", "transpose", "log_softmax", "block_backward"))
    dtype = rng.choice(("f32", "f16", "bf16"))
    step = rng.choice((1, 8, 8, 64))   # odd widths, widths of whole vectors, and the usual multiples of 64
    if kind == "softmax":
        cols = _log(rng, 16, 8192, step)
        return {"kind": kind, "rows": _rows(rng, cols, 65536, 1 << 26), "cols": cols, "dtype": dtype}
    if kind == "pack":
        return {"kind": kind, "each": rng.randint(1, 8), "rows": _log(rng, 8, 128), "cols": _log(rng, 64, 256, step)}
    if kind == "scores":
        k_len = _log(rng, 16, 1024, step)
        heads = rng.choice((8, 12, 16))
        q_len = rng.choice((1, k_len, k_len, k_len))   # one query while decoding, as many as keys otherwise
        batch = _log(rng, 1, max(1, min(128, (1 << 26) // (heads * q_len * k_len))))
        return {"kind": kind, "batch": batch, "heads": heads, "q_len": q_len, "k_len": k_len, "dtype": dtype}
    if kind in ("layernorm", "layernorm_backward", "rmsnorm", "rmsnorm_backward"):
        cols = _log(rng, 64, 8192, step)
        case = {"kind": kind, "rows": _rows(rng, cols, 65536, 1 << 25), "cols": cols, "dtype": dtype}
        if kind == "layernorm":
            case["out"] = "bf16" if dtype == "f32" else dtype
        return case
    if kind == "gelu_dbias":
        cols = _log(rng, 128, 12288, step)
        return {"kind": kind, "rows": _rows(rng, cols, 65536, 1 << 26), "cols": cols, "dtype": dtype}
    if kind == "transpose_chain":
        heads, dim, seq = rng.choice((8, 12, 16)), rng.choice((32, 64, 80, 128)), _log(rng, 16, 1024)
        return {"kind": kind, "batch": _log(rng, 1, max(1, min(64, (1 << 25) // (heads * dim * seq)))), "seq": seq, "heads": heads, "dim": dim,
                "dtype": dtype}
    if kind == "transpose":
        perm = rng.choice(("10", "021", "021", "0213", "0231", "0312"))
        d0 = _log(rng, 64, 4096, step) if perm == "10" else _log(rng, 1, 64)
        d1, d2, d3 = _log(rng, 64, 4096, step), 1, 1
        if len(perm) >= 3:
            d1, d2 = _log(rng, 16, 1024, step), _log(rng, 64, 1024, rng.choice((1, 8, 64)))
        if len(perm) == 4:
            d1, d2, d3 = _log(rng, 16, 512), rng.choice((8, 12, 16)), rng.choice((32, 64, 80, 128))
        return {"kind": kind, "d0": d0, "d1": d1, "d2": d2, "d3": d3, "perm": perm, "dtype": dtype}
    if kind == "log_softmax":
        cols = _log(rng, 8192, 131072, step)
        return {"kind": kind, "rows": _rows(rng, cols, 4096, 1 << 28), "cols": cols, "dtype": dtype}
    heads, dim = rng.choice((4, 8, 12)), rng.choice((32, 64))
    return {"kind": kind, "batch": _log(rng, 2, 32), "seq": _log(rng, 16, 256, rng.choice((1, 8))), "heads": heads, "dim": dim,
            "ffn": 4 * heads * dim, "dtype": rng.choice(("f16", "bf16"))}


# ---- descriptors and inputs ------------------------------------------------------------------------------------------
def _members(case):
    """The tiny subgraphs of a pack, `each` of three kinds and half as many of two others."""
    n, r, c = case["each"], case["rows"], case["cols"]
    half = max(1, n // 2)
    return ([W.softmax_graph(r, c, "f32")] * n + [W.add_bias_layernorm_graph(2 * r, 6 * c)] * n
            + [W.softmax_backward_graph(6 * r, c, "f16")] * n + [W.rmsnorm_graph(r, 8 * c, dtype="bf16")] * half
            + [W.bias_gelu_graph(r, 24 * c, "bf16")] * half)


def _perm(case):
    return tuple(int(p) for p in case["perm"])


def _dims(case):
    return tuple(case["d%d" % i] for i in range(len(case["perm"])))


def _specs(case):
    kind = case["kind"]
    if kind == "pack":
        return _members(case)
    if kind in ("softmax", "log_softmax"):
        return [(W.softmax_graph if kind == "softmax" else W.log_softmax_graph)(case["rows"], case["cols"], case["dtype"])]
    if kind == "scores":
        return [W.attention_scores_graph(case["batch"], case["heads"], case["q_len"], case["k_len"], dtype=case["dtype"])]
    if kind == "layernorm":
        return [W.add_bias_layernorm_graph(case["rows"], case["cols"], in_dtype=case["dtype"], out_dtype=case["out"])]
    if kind == "layernorm_backward":
        return [W.layernorm_backward_graph(case["rows"], case["cols"], case["dtype"])]
    if kind == "rmsnorm":
        return [W.rmsnorm_graph(case["rows"], case["cols"], dtype=case["dtype"])]
    if kind == "rmsnorm_backward":
        return [W.rmsnorm_backward_graph(case["rows"], case["cols"], case["dtype"])]
    if kind == "gelu_dbias":
        return [W.bias_gelu_dbias_graph(case["rows"], case["cols"], case["dtype"])]
    if kind == "transpose_chain":
        return [W.transpose_chain_graph(case["batch"], case["seq"], case["heads"], case["dim"], dtype=case["dtype"])]
    if kind == "transpose":
        return [W.transpose_graph(_dims(case), _perm(case), case["dtype"])]
    if kind == "block_backward":
        return [W.transformer_block_backward_graph(case["batch"], case["seq"], case["heads"], case["dim"], case["ffn"], case["dtype"])]
    raise ValueError(kind)


def _inputs(spec, seed):
    """Activations and gradients ~ N(0,1), scores ~ N(0,3), gains ~ 1 + N(0,0.02), biases ~ N(0,0.02), saved means
    ~ N(0,0.05) and reciprocal deviations ~ U(0.8,1.2), probabilities whose rows sum to 1, additive masks of 0 and
    -10000 from per-sequence valid lengths."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    out = {}
    for t in spec.inputs:
        n = t.name
        if n == "mask":
            lens = torch.randint(min(16, t.dims[-1]), t.dims[-1] + 1, (t.dims[0], 1, 1, 1), generator=g, device=DEVICE)
            a = torch.where(torch.arange(t.dims[-1], device=DEVICE) < lens, 0.0, -10000.0)
        elif n in ("y", "probs"):
            a = torch.empty(t.dims, device=DEVICE).exponential_(generator=g)
            a /= a.sum(-1, keepdim=True)
        elif n.startswith("rstd") or n in ("rrms", "scale"):
            a = torch.empty(t.dims, device=DEVICE).uniform_(0.8, 1.2, generator=g)
        else:
            a = torch.randn(t.dims, generator=g, device=DEVICE)
            if n == "scores":
                a *= 3.0
            elif n == "g" and len(t.dims) == 1 or n.startswith("gamma"):
                a = 1.0 + 0.02 * a
            elif n.startswith(("bias", "beta")):
                a *= 0.02
            elif n.startswith("mu"):
                a *= 0.05
        out[n] = a.to(DTYPE[t.dtype])
    return out


def prepare(case, seed):
    specs = _specs(case)
    ins = [_inputs(s, 1000 * seed + i) for i, s in enumerate(specs)]
    tensors = [d[t.name] for s, d in zip(specs, ins) for t in s.inputs]
    outs = [B.alloc_outputs(s) for s in specs]
    flat = [t for o in outs for t in o]
    stream = torch.cuda.current_stream().cuda_stream
    in_ptrs, out_ptrs = [t.data_ptr() for t in tensors], [t.data_ptr() for t in flat]
    ws = None
    if case["kind"] == "pack":
        plans = [B.Plan(B.Graph.from_spec(s)) for s in specs]
        what = B.Pack(plans)
        call = what.bind(in_ptrs, out_ptrs, stream)
    else:
        graph = B.Graph.from_spec(specs[0])
        what = B.Program(graph) if case["kind"] == "block_backward" else B.Plan(graph)
        ws = what.make_workspace()
        call = what.bind(in_ptrs, out_ptrs, ws.data_ptr() if ws is not None else 0, ws.numel() if ws is not None else 0, stream)
    return {"call": call, "outputs": flat, "keep": (what, tensors, ws)}


def run(state):
    state["call"]()
    return state["outputs"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
OPS_PER_ELEMENT = {"softmax": 5, "log_softmax": 5, "scores": 7, "layernorm": 9, "layernorm_backward": 16, "rmsnorm": 4, "rmsnorm_backward": 10,
                   "gelu_dbias": 20, "transpose_chain": 4, "transpose": 0, "pack": 6, "block_backward": 12}


def work(case):
    """Every input read once, every output written once; operations per element of the largest input."""
    size = ops = 0
    for s in _specs(case):
        shapes = B.output_shapes(s)
        size += sum(math.prod(t.dims) * SIZE[t.dtype] for t in s.inputs) + sum(math.prod(shapes[n]) * SIZE[d] for n, d in s.outputs)
        ops += max(math.prod(t.dims) for t in s.inputs) * OPS_PER_ELEMENT[case["kind"]]
    return {"bytes": size, "flops": ops}


def tolerance(case):
    """Arithmetic is float32 throughout.  Outputs stored in 16 bits are off by their own rounding (2-norm measured against
    `exact`: 1.7e-3 in bfloat16, 2.1e-4 in float16) and by ties that fall the other way; outputs stored in float32 by
    their arithmetic (measured: rows up to 1e-7; column sums over tens of thousands of rows up to 8e-7, by the order of
    the sum).  Stated is about four times that."""
    kind = case["kind"]
    if kind == "transpose":
        return "exact"
    stored = case.get("out", case.get("dtype", "bf16"))
    return {"rel": {"f32": 4e-6 if kind in ("layernorm_backward", "rmsnorm_backward", "gelu_dbias") else 1e-6, "f16": 8e-4, "bf16": 7e-3}[stored]}


# ---- the same in float64 ---------------------------------------------------------------------------------------------
def _round(x, dtype):
    return x if dtype == "f32" else x.to(DTYPE[dtype]).double()


def _gelu(z):
    """tanh-GELU and its derivative."""
    k = math.sqrt(2.0 / math.pi)
    t = torch.tanh(k * (z + 0.044715 * z ** 3))
    return 0.5 * z * (1.0 + t), 0.5 * (1.0 + t) + 0.5 * z * (1.0 - t * t) * k * (1.0 + 3 * 0.044715 * z * z)


def _norm_backward(h, mu, rstd, dy, gamma):
    xh = (h - mu) * rstd
    g = dy * gamma
    dx = rstd * (g - g.mean(1, keepdim=True) - xh * (g * xh).mean(1, keepdim=True))
    return dx, (dy * xh).sum(0, keepdim=True), dy.sum(0, keepdim=True)


def _block_backward(v, case):
    """The block's gradients; values that the graph rounds to the storage dtype are rounded here too, since later ops
    read the rounded ones."""
    dt = case["dtype"]
    dx2, dg2, db2 = _norm_backward(v["h2"], v["mu2"], v["rstd2"], v["dy2"], v["gamma2"])
    dx2 = _round(dx2, dt)
    f = _round(v["up_act"] * _gelu(v["ffn1_pre"] + v["bias1"])[1], dt)
    dx1, dg1, db1 = _norm_backward(v["h1"], v["mu1"], v["rstd1"], dx2 + v["up_l1"], v["gamma1"])
    dx1 = _round(dx1, dt)
    p, dp = v["probs"], v["up_probs"]
    ds = p * (dp - (p * dp).sum(-1, keepdim=True)) * float(case["dim"]) ** -0.5
    col = lambda x: x.sum(0, keepdim=True)  # noqa: E731
    swap = lambda x: x.transpose(1, 2).contiguous()  # noqa: E731
    return [dx2, dg2, db2, col(dx2), f, col(f), dx1, dg1, db1, col(dx1), swap(v["up_ctx"]), ds, swap(v["up_q"]), swap(v["up_k"]), swap(v["up_v"])]


def _exact(spec, kind, case, v):
    if kind in ("softmax", "log_softmax"):
        return [(torch.softmax if kind == "softmax" else torch.log_softmax)(v["x"], -1)]
    if kind == "scores":
        return [torch.softmax(v["scores"] * 0.125 + v["mask"], -1)]
    if kind == "layernorm":
        h = v["x"] + v["res"] + v["bias"]
        c = h - h.mean(1, keepdim=True)
        return [c * torch.rsqrt((c * c).mean(1, keepdim=True) + 1e-5) * v["gamma"] + v["beta"]]
    if kind == "layernorm_backward":
        return list(_norm_backward(v["h"], v["mu"], v["rstd"], v["dy"], v["gamma"]))
    if kind == "rmsnorm":
        return [v["x"] * torch.rsqrt((v["x"] * v["x"]).mean(1, keepdim=True) + 1e-6) * v["gamma"]]
    if kind == "rmsnorm_backward":
        xh = v["x"] * v["rrms"]
        gy = v["dy"] * v["g"]
        return [(gy - xh * (gy * xh).mean(1, keepdim=True)) * v["rrms"], (v["dy"] * xh).sum(0, keepdim=True)]
    if kind == "softmax_backward":
        return [v["y"] * (v["dy"] - (v["y"] * v["dy"]).sum(1, keepdim=True))]
    if kind == "bias_gelu":
        return [_gelu(v["x"] + v["bias"])[0]]
    if kind == "gelu_dbias":
        y, d = _gelu(v["x"] + v["bias"])
        return [y, (v["grad"] * d).sum(0, keepdim=True)]
    if kind == "transpose_chain":
        u = v["x"].transpose(1, 2) * v["scale"]
        return [(u * torch.rsqrt((u * u).sum(-1, keepdim=True) + 1e-6)).contiguous()]
    if kind == "block_backward":
        return _block_backward(v, case)
    raise ValueError(kind)


def exact(case, seed):
    specs = _specs(case)
    out = []
    for i, s in enumerate(specs):
        v = _inputs(s, 1000 * seed + i)
        kind = case["kind"]
        if kind == "transpose":   # moved bits: compared in their own type
            out.append(v["x"].permute(_perm(case)).contiguous())
            continue
        if kind == "pack":
            kind = {"softmax_b": "softmax_backward", "softmax_f": "softmax", "add_bias_": "layernorm", "rmsnorm_b": "rmsnorm", "bias_gelu": "bias_gelu"}[s.name[:9]]
        out += _exact(s, kind, case, {n: t.double() for n, t in v.items()})
    return out
