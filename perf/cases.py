"""Performance cases: what a serving program asks of this library, from the smallest call to the largest.

A case is a dict of plain values.  Three kinds:

  linear  the linear layers of a model at one batch size: `shapes` ("NxK NxK ..."), repeated for
          `layers` model layers, each quantising its FP16 activations (`quantize`, with smooth
          scales where `smooth`) and multiplying them with its packed weights.  `graph`: captured
          once and replayed, as serving programs run their decode steps; otherwise one Python call
          after the other, as they run prefill.
  moe     a mixture-of-experts feed-forward layer: tokens sorted by expert, quantised, grouped up
          projection, quantised, grouped down projection.
  quant   the activation quantisation alone.

Weights are Gaussian FP16 matrices quantised by the library's packer; activations are Gaussian FP16
with, where `outliers`, one channel in a thousand twenty times as large.  The attention and the
activation function between two layers are not this library's work: every layer gets activations
of its own.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_01229_amd import api

DEVICE = "cuda"


def listed():
    return [
        # one token through one projection from Python: launches and host work are all there is
        _linear("call_m1", 1, "4096x4096", 64, graph=False),
        # a decode step of a few users on a 7B model: four projections in each of two layers
        _linear("decode_7b_m4", 4, "4096x4096 4096x4096 11008x4096 4096x11008", 64, layers=2),
        # a decode step on a 70B model: the weights stream from HBM
        _linear("decode_70b_m16", 16, "10240x8192 28672x8192 8192x28672", 128),
        # a decode step of several dozen users (a ragged number of them) on a 13B model
        _linear("decode_13b_m45", 45, "5120x5120 13824x5120 5120x13824", 64, layers=2),
        # a large decode batch, or a short prompt, on a 7B model's feed-forward layers
        _linear("mlp_7b_m128", 128, "11008x4096 4096x11008", 64, layers=2, outliers=True),
        # a chunk of a chunked prefill on a 70B model's attention projections, smooth scales applied on the fly
        _linear("chunk_70b_m256", 256, "10240x8192 8192x8192", 128, smooth=True),
        # a prompt of odd length through a 7B model's feed-forward layers (K = 11008 is no multiple of 512)
        _linear("prompt_7b_m509", 509, "11008x4096 4096x11008", 64, graph=False, outliers=True),
        # prefill on activations that are quantised already: one round of tiles, then the large GEMM
        _linear("prefill_m1024", 1024, "8192x8192", 64, graph=False, quantize=False),
        _linear("prefill_m4096", 4096, "8192x8192", 64, graph=False, quantize=False),
        # mixture-of-experts layers of 8 experts: a decode batch (about 16 rows an expert) and a prompt
        _moe("moe_decode_t64", 64, 8, 14336, 4096, 64),
        _moe("moe_prefill_t3000", 3000, 8, 14336, 4096, 64),
        # the quantisation of a long prompt with smooth scales
        _quant("quant_smooth_m4096", 4096, 8192, smooth=True),
    ]


def _linear(name, M, shapes, group, layers=1, graph=True, quantize=True, smooth=False, outliers=False):
    c = dict(name=name, kind="linear", M=M, shapes=shapes, group=group, layers=layers, graph=graph,
             quantize=quantize, smooth=smooth, outliers=outliers)
    return c if name else _unnamed(c)


def _moe(name, tokens, experts, inter, hidden, group):
    c = dict(name=name, kind="moe", tokens=tokens, experts=experts, top_k=2, inter=inter, hidden=hidden, group=group)
    return c if name else _unnamed(c)


def _quant(name, M, K, smooth):
    c = dict(name=name, kind="quant", M=M, K=K, smooth=smooth)
    return c if name else _unnamed(c)


def _unnamed(c):
    del c["name"]
    return c


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: a layer of any width, depth and batch size of the ranges above."""
    pick = rng.random()
    if pick < 0.70:
        M = _log_int(rng, 1, 4096)
        N, K = 64 * _log_int(rng, 16, 448), 256 * _log_int(rng, 8, 112)
        while M * N * K > 4096 * 8192 * 8192:  # no more than the largest GEMM above
            N, K = 64 * _log_int(rng, 16, 448), 256 * _log_int(rng, 8, 112)
        decode = M <= 256  # replayed from a graph, four layers of it; prefill is called
        return _linear("", M, f"{N}x{K}", rng.choice((64, 128)), layers=4 if decode else 1, graph=decode,
                       quantize=decode or rng.random() < 0.5, smooth=rng.random() < 0.25, outliers=rng.random() < 0.5)
    if pick < 0.85:
        inter, hidden = 256 * _log_int(rng, 8, 56), 256 * _log_int(rng, 8, 20)
        return _moe("", _log_int(rng, 4, 3000), rng.choice((4, 8, 16)), inter, hidden, rng.choice((64, 128)))
    return _quant("", _log_int(rng, 16, 8192), 8 * _log_int(rng, 256, 2048), smooth=rng.random() < 0.5)


# ----------------------------------------------------------------------------- inputs
def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split()] * case["layers"]


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _weights_f16(N, K, gen):
    return torch.randn((N, K), generator=gen, device=DEVICE, dtype=torch.float32).mul_(0.02).to(torch.float16)


def _activations_f16(M, K, gen, outliers):
    X = torch.randn((M, K), generator=gen, device=DEVICE, dtype=torch.float32)
    if outliers:
        X[:, torch.randperm(K, generator=gen, device=DEVICE)[: max(1, K // 1000)]] *= 20.0
    return X.to(torch.float16)


def _smooth(K, gen):
    return torch.exp(torch.randn((K,), generator=gen, device=DEVICE, dtype=torch.float32) * 0.5)


def _pack(W, group):
    return tuple(torch.from_numpy(t).to(DEVICE) for t in api.liquidquant_pack_weights(W.cpu().numpy(), group))


def _row_offsets(case, seed):
    """Rows of each expert (top_k experts a token, all equally likely), as running totals."""
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = rng.multinomial(case["tokens"] * case["top_k"], [1.0 / case["experts"]] * case["experts"])
    return [0] + [int(r) for r in np.cumsum(rows)]


# (the inputs of a case, drawn in one order; exact() draws the same)
def _linear_inputs(case, seed):
    gen = _generator(seed)
    for N, K in _shapes(case):
        W = _weights_f16(N, K, gen)
        X = _activations_f16(case["M"], K, gen, case["outliers"])
        yield N, K, W, X, _smooth(K, gen) if case["smooth"] else None


def _moe_inputs(case, seed):
    """Per projection: N, K, the weights (the experts share their integers and differ in their
    channel scales, so that making them stays quick), the experts' scale factors, the activations."""
    gen = _generator(seed)
    rows, E = case["tokens"] * case["top_k"], case["experts"]
    for N, K in ((case["inter"], case["hidden"]), (case["hidden"], case["inter"])):
        W = _weights_f16(N, K, gen)
        factors = torch.rand((E, 1), generator=gen, device=DEVICE, dtype=torch.float32) + 0.5
        yield N, K, W, factors, _activations_f16(rows, K, gen, False)


def _quant_inputs(case, seed):
    gen = _generator(seed)
    return _activations_f16(case["M"], case["K"], gen, True), _smooth(case["K"], gen) if case["smooth"] else None


def prepare(case, seed):
    if case["kind"] == "quant":
        X, smooth = _quant_inputs(case, seed)
        return {"call": lambda: list(api.w4a8_quantize_activations(X, smooth))}
    if case["kind"] == "moe":
        return _prepare_moe(case, seed)
    return _prepare_linear(case, seed)


def _prepare_linear(case, seed):
    group, M = case["group"], case["M"]
    layers = []
    for N, K, W, X, smooth in _linear_inputs(case, seed):
        packed = _pack(W, group)
        layers.append((N, K, packed, X if case["quantize"] else api.w4a8_quantize_activations(X, smooth), smooth))

    def step(workspace=None):
        out = []
        for N, K, packed, x, smooth in layers:
            q, scales = api.w4a8_quantize_activations(x, smooth) if case["quantize"] else x
            out.append(api.w4a8_gemm(q, scales, *packed, N, K, group, workspace=workspace))
        return out

    if not case["graph"]:
        return {"call": step}
    need = max(api.w4a8_gemm_workspace_size(M, N, K, group) for N, K in _shapes(case))
    workspace = torch.empty(max(need, 16), dtype=torch.uint8, device=DEVICE)
    api.w4a8_workspace_init(workspace)
    step(workspace)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = step(workspace)
    return {"graph": graph, "out": out, "keep": (layers, workspace)}


def _prepare_moe(case, seed):
    offsets, group, E = _row_offsets(case, seed), case["group"], case["experts"]
    projections = []
    for N, K, W, factors, X in _moe_inputs(case, seed):
        codes, gparams, scales = _pack(W, group)
        projections.append((N, K, codes.repeat(E), gparams.repeat(E), (scales * factors).contiguous(), X))

    def layer():
        out = []
        for N, K, codes, gparams, scales, x in projections:
            q, sx = api.w4a8_quantize_activations(x)
            out.append(api.w4a8_grouped_gemm(offsets, q, sx, codes, gparams, scales, N, K, group)[0])
        return out

    return {"call": layer}


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return state["call"]()


# ------------------------------------------------------------------- what a pass cannot do without
def _gemm_work(M, N, K, group, x_bytes, experts=1):
    weights = experts * (N * K // 2 + 2 * N * K // group + 4 * N)
    return weights + M * K * x_bytes + 2 * M * N, 2 * M * N * K


def work(case):
    if case["kind"] == "quant":
        M, K = case["M"], case["K"]
        return {"bytes": 3 * M * K + 4 * M + (4 * K if case["smooth"] else 0), "flops": 4 * M * K}
    if case["kind"] == "moe":
        rows, N, K = case["tokens"] * case["top_k"], case["inter"], case["hidden"]
        parts = [_gemm_work(rows, n, k, case["group"], 2, min(case["experts"], rows)) for n, k in ((N, K), (K, N))]
    else:
        x_bytes = 2 if case["quantize"] else 1
        parts = [_gemm_work(case["M"], n, k, case["group"], x_bytes) for n, k in _shapes(case)]
        parts += [(4 * k, 0) for _, k in _shapes(case) if case["smooth"] and case["quantize"]]
        parts += [(4 * case["M"], 0) for _ in _shapes(case) if not case["quantize"]]
    return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}


def tolerance(case):
    """The integer product is exact and each output is rounded to FP16 once or twice (half a unit in
    the last place is 4.9e-4 of the value; against exact() the path is 2.1e-4 off in the 2-norm).
    The quantisation is defined bit for bit."""
    return "exact" if case["kind"] == "quant" else {"rel": 1e-3, "max": 2e-3}


# ----------------------------------------------------------------------------- the same in 64 bits
def _f32(v):
    return v.to(torch.float32).to(torch.float64)


def _exact_quantize(X, smooth):
    x = X.double()
    if smooth is not None:
        x = _f32(x / smooth.double())
    amax = x.abs().amax(dim=1, keepdim=True)
    s = torch.where(amax > 0, _f32(amax / 127.0), torch.ones_like(amax))
    return torch.clamp(torch.round(_f32(x / s)), -127, 127), s


def _exact_weights(W, group):
    """Two-level LiquidQuant quantisation: dequantised level-1 integers and the channel scales."""
    w = W.double()
    amax = w.abs().amax(dim=1, keepdim=True)
    s_w = torch.where(amax > 0, _f32(amax / 119.0), torch.ones_like(amax))
    q = torch.clamp(torch.round(_f32(w / s_w)), -119, 119).view(W.shape[0], -1, group)
    low = q.amin(dim=2, keepdim=True)
    s = torch.clamp(torch.floor((2 * (q.amax(dim=2, keepdim=True) - low) + 15) / 30), min=1)
    code = torch.clamp(torch.floor((2 * (q - low) + s) / (2 * s)), max=15)
    return (code * s + low).view(W.shape), s_w[:, 0]


def exact(case, seed):
    if case["kind"] == "quant":
        q, s = _exact_quantize(*_quant_inputs(case, seed))
        return [q.to(torch.int8), s[:, 0]]
    out = []
    if case["kind"] == "moe":
        offsets = _row_offsets(case, seed)
        for N, K, W, factors, X in _moe_inputs(case, seed):
            q, s = _exact_quantize(X, None)
            wd, s_w = _exact_weights(W, case["group"])
            y = torch.matmul(q, wd.t()) * s
            for e in range(case["experts"]):
                y[offsets[e] : offsets[e + 1]] *= _f32(s_w * factors[e].double())
            out.append(y)
    else:
        for N, K, W, X, smooth in _linear_inputs(case, seed):
            q, s = _exact_quantize(X, smooth)
            wd, s_w = _exact_weights(W, case["group"])
            out.append(torch.matmul(q, wd.t()) * s * s_w)
    return out
