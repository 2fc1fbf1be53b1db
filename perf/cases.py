"""The workloads that the few-bit activation's speed is judged by.

A case is one pass of a user's program through the public entry points:

  mode "module"  a training step through the drop-in layer FewBitAct: the
                 forward under autograd and the gradient of its input;
  mode "calls"   fwd and bwd called directly, each allocating its results (a
                 program with an autograd function of its own);
  mode "kept"    the same two calls into buffers that the program keeps;
  mode "fwd"     the forward alone into kept buffers (recomputation in
                 checkpointed training, where codes are written afresh);
  mode "bwd"     the backward alone into a kept buffer;
  mode "graph"   a HIP graph with the forwards and then, in reverse order, the
                 backwards of a stack of layers, replayed.

The fitted table belongs to the program's set-up (one per activation, bit
width and weight) and is kept; inputs and gradients differ by seed.
"""
from __future__ import annotations

import functools
import math

import torch

import paper_2202_00441_amd as P

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
DISTRIBUTIONS = ("normal", "wide", "outliers", "uniform")


def _case(name, mode, act, bits, dtype, n, dist, symmetric=False, layers=1):
    c = {"mode": mode, "act": act, "bits": bits, "dtype": dtype, "n": n, "dist": dist,
         "symmetric": symmetric, "layers": layers}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # a fine-tuning step on a handful of tokens (32 x 3072): launches and host work only
        _case("module_bf16_gelu3_32x3072", "module", "gelu", 3, "bf16", 32 * 3072, "normal"),
        # the largest ragged size of the parity sweep, fp16, direct calls
        _case("calls_f16_tanh4_100003", "calls", "tanh", 4, "f16", 100003, "normal", symmetric=True),
        # the 1M-element fp32 vector of the workload list
        _case("calls_f32_gelu3_1m", "calls", "gelu", 3, "f32", 1 << 20, "normal"),
        # the 12 feed-forward activations of a small language model at 256 tokens,
        # captured in a graph because each one is far shorter than a launch from the host
        _case("graph_bf16_gelu3_12x256x3072", "graph", "gelu", 3, "bf16", 256 * 3072, "normal", layers=12),
        # four BERT-base feed-forward activations at 8 x 512 tokens, in a captured step
        _case("graph_bf16_gelu3_4x8x512x3072", "graph", "gelu", 3, "bf16", 8 * 512 * 3072, "wide", layers=4),
        # a ResNet stage with SiLU in fp16 at 2 bits
        _case("calls_f16_silu2_64x256x56x56", "calls", "silu", 2, "f16", 64 * 256 * 56 * 56, "normal"),
        # recomputing forward, fp16 GELU at 4 bits, 2^26 elements (the size of the benchmark's sweep)
        _case("fwd_f16_gelu4_64m", "fwd", "gelu", 4, "f16", 1 << 26, "wide"),
        # self-normalising network in bf16, an odd length between the powers of two
        _case("calls_bf16_selu2_odd_34m", "calls", "selu", 2, "bf16", 33_950_117, "normal"),
        # the two long odd fp32 vectors of the workload list
        _case("calls_f32_sigmoid4_odd_67m", "calls", "sigmoid", 4, "f32", 67_108_863, "uniform", symmetric=True),
        _case("module_f32_tanh3_odd_67m", "module", "tanh", 3, "f32", 67_108_863, "uniform"),
        # the feed-forward activation of a large language model, 16 x 2048 x 8192: the headline
        _case("module_bf16_gelu3_16x2048x8192", "module", "gelu", 3, "bf16", 16 * 2048 * 8192, "outliers"),
        # the same at 1 bit into kept buffers
        _case("kept_bf16_gelu1_16x2048x8192", "kept", "gelu", 1, "bf16", 16 * 2048 * 8192, "outliers"),
    ]


# no drawn case moves more bytes than the largest listed one
_MOST_BYTES = 2 * 4.375 * (16 * 2048 * 8192)


def draw(rng):
    mode = rng.choice(("module", "module", "calls", "kept", "fwd", "bwd", "graph"))
    act = rng.choice(("gelu", "gelu", "silu", "silu", "sigmoid", "tanh", "relu", "selu", "softplus"))
    bits = rng.choice((1, 2, 3, 3, 4))
    dtype = rng.choice(("f32", "f16", "bf16", "bf16"))
    symmetric = act in ("sigmoid", "tanh") and rng.random() < 0.5
    layers = rng.choice((4, 8, 12)) if mode == "graph" else 1
    top = {1: 28.0, 4: 24.0}.get(layers, 20.0)
    n = int(2.0 ** rng.uniform(11.0, top))
    if rng.random() < 0.5:                 # whole rows of a model's width
        n = max(1, n // 768) * 768
    elif n % 2 == 0:
        n += 1
    c = _case(None, mode, act, bits, dtype, n, rng.choice(DISTRIBUTIONS), symmetric, layers)
    over = work(c)["bytes"] / _MOST_BYTES
    if over > 1.0:
        c["n"] = int(n / over) - 1
    return c


# ---------------------------------------------------------------- inputs
@functools.lru_cache(maxsize=None)
def _table(act, bits, symmetric):
    """The fitted table: standard normal weight on [-10, 10], 4000 cells, as
    FewBitAct fits it by default.  It is data of the operation, as weights are,
    for the reference values below too."""
    return P.fit_table(act, bits, P.Weight(P.W_NORMAL, -10.0, 10.0), 4000, symmetric=symmetric)


def _inputs(case, seed):
    """x and grad_out of every layer, drawn on the GPU from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt, n = DTYPES[case["dtype"]], case["n"]
    pairs = []
    for _ in range(case["layers"]):
        if case["dist"] == "uniform":
            x = torch.rand(n, generator=gen, device="cuda").mul_(16.0).sub_(8.0)
        else:
            x = torch.randn(n, generator=gen, device="cuda")
            if case["dist"] == "wide":
                x.mul_(1.5)
            elif case["dist"] == "outliers":          # 1% of the values ten times as large
                x.mul_((torch.rand(n, generator=gen, device="cuda") < 0.01).mul(9.0).add_(1.0))
        x = x.to(dt)
        g = torch.randn(n, generator=gen, device="cuda").to(dt)
        pairs.append((x, g))
    return pairs


def _codes_buffer(n, bits):
    return torch.empty(P.packed_words(n, bits), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    table = _table(case["act"], case["bits"], case["symmetric"])
    pairs = _inputs(case, seed)
    mode, n, bits = case["mode"], case["n"], case["bits"]
    state = {"mode": mode, "table": table, "x": pairs[0][0], "g": pairs[0][1]}
    x, g = pairs[0]
    if mode == "module":
        state["layer"] = P.FewBitAct(case["act"], bits, table=table)
        x.requires_grad_()
    elif mode in ("kept", "fwd"):
        state["y"], state["codes"] = torch.empty_like(x), _codes_buffer(n, bits)
        state["grad"] = torch.empty_like(x) if mode == "kept" else None
    elif mode == "bwd":
        state["codes"] = P.fwd(table, x)[1]
        state["grad"] = torch.empty_like(g)
    elif mode == "graph":
        layers = [{"x": x, "g": g, "y": torch.empty_like(x), "codes": _codes_buffer(n, bits),
                   "grad": torch.empty_like(g)} for x, g in pairs]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _stack(table, layers)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _stack(table, layers)
        state["layers"], state["graph"] = layers, graph
    return state


def _stack(table, layers):
    for s in layers:
        P.fwd(table, s["x"], s["y"], s["codes"])
    for s in reversed(layers):
        P.bwd(table, s["g"], s["codes"], s["grad"])


# ---------------------------------------------------------------- one pass
def run(state):
    mode, table = state["mode"], state["table"]
    if mode == "module":
        y = state["layer"](state["x"])
        (grad,) = torch.autograd.grad(y, state["x"], state["g"])
        return {"y": y, "grad": grad}
    if mode == "calls":
        y, codes = P.fwd(table, state["x"])
        return {"y": y, "codes": codes, "grad": P.bwd(table, state["g"], codes)}
    if mode == "kept":
        P.fwd(table, state["x"], state["y"], state["codes"])
        P.bwd(table, state["g"], state["codes"], state["grad"])
        return {"y": state["y"], "codes": state["codes"], "grad": state["grad"]}
    if mode == "fwd":
        P.fwd(table, state["x"], state["y"], state["codes"])
        return {"y": state["y"], "codes": state["codes"]}
    if mode == "bwd":
        return {"grad": P.bwd(table, state["g"], state["codes"], state["grad"])}
    state["graph"].replay()
    return [{k: s[k] for k in ("y", "codes", "grad")} for s in state["layers"]]


# ---------------------------------------------------------------- what a pass needs
def work(case):
    n, s, bits = case["n"], SIZE[case["dtype"]], case["bits"]
    one_way = 2 * n * s + 4 * ((n * bits + 31) // 32)
    directions = 1 if case["mode"] in ("fwd", "bwd") else 2
    # per element: f (about ten operations) and bits compares forward, one product backward
    flops = {"fwd": 10 + bits, "bwd": 1}.get(case["mode"], 11 + bits)
    return {"bytes": case["layers"] * directions * one_way, "flops": case["layers"] * n * flops}


def tolerance(case):
    # Codes are whole numbers and stay the same.  y and the gradient are one
    # rounding to the storage type away from an fp32 evaluation: about four
    # times the distance from 64 bits that the path shows.
    return {"rel": {"f32": 1e-6, "f16": 9e-4, "bf16": 7e-3}[case["dtype"]]}


# ---------------------------------------------------------------- reference
_LAMBDA, _ALPHA = 1.0507009873554805, 1.6732632423543772


def _f(act, x):
    if act == "gelu":
        return 0.5 * x * torch.special.erfc(x * -math.sqrt(0.5))
    if act == "silu":
        return x * torch.sigmoid(x)
    if act == "sigmoid":
        return torch.sigmoid(x)
    if act == "tanh":
        return torch.tanh(x)
    if act == "relu":
        return torch.clamp(x, min=0.0)
    if act == "selu":
        return torch.where(x > 0, _LAMBDA * x, _LAMBDA * _ALPHA * torch.expm1(x))
    return torch.clamp(x, min=0.0) + torch.log1p(torch.exp(-x.abs()))


def _exact_one(case, x, g):
    bits, n, chunk = case["bits"], case["n"], 1 << 25         # whole words at every bit width
    table = _table(case["act"], bits, case["symmetric"])
    s = torch.tensor(table.s, dtype=torch.float64, device="cuda")
    v = torch.tensor(table.v, dtype=torch.float64, device="cuda")
    y, grad, words = [], [], []
    for at in range(0, n, chunk):
        xd = x[at:at + chunk].double()
        idx = torch.searchsorted(s, xd.abs() if case["symmetric"] else xd, right=True)
        y.append(_f(case["act"], xd))
        grad.append(g[at:at + chunk].double() * v[idx])
        stream = (idx.unsqueeze(1) >> torch.arange(bits, device="cuda")).bitwise_and_(1).to(torch.uint8).reshape(-1)
        stream = torch.nn.functional.pad(stream, (0, -stream.numel() % 32)).reshape(-1, 32)
        low = torch.zeros(stream.shape[0], dtype=torch.int64, device="cuda")
        for b in range(32):
            low |= stream[:, b].to(torch.int64) << b
        words.append(torch.where(low >= 1 << 31, low - (1 << 32), low).to(torch.int32))
    return {"y": torch.cat(y), "codes": torch.cat(words), "grad": torch.cat(grad)}


def exact(case, seed):
    outs = [_exact_one(case, x, g) for x, g in _inputs(case, seed)]
    if case["mode"] == "graph":
        return outs
    keep = {"module": ("y", "grad"), "fwd": ("y", "codes"), "bwd": ("grad",)}.get(case["mode"], ("y", "codes", "grad"))
    return {k: outs[0][k] for k in keep}
