"""The work that users of this library have it do, as cases that can be timed
and checked.

A case is one call, or one layer's calls, through the public entry points of
`paper_2508_02343_amd.binding`:

  linear   bf16 activations -> quantize_act (or, with norm, rmsnorm_quantize_act)
           -> gemm against a weight quantised beforehand
  layer    the four linear layers of one decoder layer at a decode step,
           captured as a HIP graph once and replayed
  weight   quantize_weight, run once per weight when a model is loaded
  calib    calibrate, run once per layer on a calibration set

Inputs follow `paper_2508_02343_amd.workloads`: normal activations with 1 % of
the channels scaled up by 30 and put last by sigma, weights N(0, 0.02).
"""

import math

import torch

from paper_2508_02343_amd import binding as B

EPS = 1e-5
OUTLIERS, OUTLIER_SCALE, W_STD = 0.01, 30.0, 0.02
LAYER = (  # (input width, output width, norm in front): QKV stacked, attention output, gate and up stacked, down
    (4096, 6144, True), (4096, 4096, False), (4096, 28672, True), (14336, 4096, False))
MAX_MNK = 8192 * 5120 * 27648


def _split(K, f4=0.75, f6=0.1875):
    p4 = round(K * f4 / 32) * 32
    p6 = min(round(K * f6 / 32) * 32, K - p4)
    return p4, p6, K - p4 - p6


def _linear(name, M, K, N, split=None, norm=False, kept=False, fp6="E3M2", fp8="E4M3"):
    p4, p6, p8 = split or _split(K)
    c = {"op": "linear", "M": M, "K": K, "N": N, "p4": p4, "p6": p6, "p8": p8, "norm": norm, "kept": kept,
         "fp6": fp6, "fp8": fp8}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one token through an attention projection, one launch at a time, into buffers that are kept: the smallest call
        _linear("decode_1_attn", 1, 4096, 4096, (2048, 1024, 1024), kept=True),
        # a decode step of eight sequences: one decoder layer's linear layers, replayed as a captured graph
        {"name": "decode_8_layer", "op": "layer", "M": 8},
        # 32 sequences, the norm and the up projection
        _linear("decode_32_up", 32, 4096, 14336, (2048, 1024, 1024), norm=True, kept=True),
        # a serving batch of 128 sequences: the norm and the stacked QKV projection
        _linear("batch_128_qkv", 128, 4096, 6144, norm=True, kept=True),
        # a ragged prompt chunk through the widest down projection (Qwen2.5-32B), buffers made by the call
        _linear("chunk_333_wide_down", 333, 27648, 5120),
        # prefill of 2048 tokens: attention projection of Llama-3-8B (the benchmark's default)
        _linear("prefill_2048_attn", 2048, 4096, 4096, (3072, 768, 256), kept=True),
        # prefill of 4096 tokens: norm and up projection of Llama-3-8B
        _linear("prefill_4096_up", 4096, 4096, 14336, norm=True, kept=True),
        # and its down projection
        _linear("prefill_4096_down", 4096, 14336, 4096, kept=True),
        # prefill of 8192 tokens: norm and up projection of Qwen2.5-32B, the largest call
        _linear("prefill_8192_wide_up", 8192, 5120, 27648, (3584, 1024, 512), norm=True, kept=True),
        # the other element formats, with ragged sizes (a vocabulary slice that is no multiple of a tile)
        _linear("formats_1000_ragged", 1000, 4096, 5400, (1024, 1536, 1536), fp6="E2M3", fp8="E5M2"),
        # a weight quantised while a model is loaded (Llama-3-8B up projection)
        {"name": "weight_14336x4096", "op": "weight", "N": 14336, "K": 4096, "p4": 3072, "p6": 768, "p8": 256,
         "fp6": "E3M2", "fp8": "E4M3"},
        # sigma and the split of one layer from 16 sequences of 2048 tokens
        {"name": "calib_32768x4096", "op": "calib", "rows": 32768, "K": 4096, "fp6": "E3M2", "fp8": "E4M3"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["linear"] * 8 + ["layer", "weight", "calib"])
    if op == "layer":
        return {"op": "layer", "M": _log(rng, 1, 256)}
    K = 32 * _log(rng, 512 // 32, 27648 // 32)
    fp6, fp8 = rng.choice([("E3M2", "E4M3")] * 4 + [("E2M3", "E5M2"), ("E2M3", "E4M3")])
    if op == "calib":
        return {"op": "calib", "rows": _log(rng, 64, min(32768, (1 << 28) // K)), "K": K, "fp6": fp6, "fp8": fp8}
    # mostly the split of about 5 bits per element, now and then one format alone or nearly even groups
    f4, f6 = rng.choice([(0.75, 0.1875)] * 2 + [(rng.uniform(0.5, 0.9), 0.1), (0.5, 0.25), (1.0, 0.0), (0.0, 0.0)])
    p4, p6, p8 = _split(K, f4, f6)
    if op == "weight":
        return {"op": "weight", "N": _log(rng, 512, min(28672, (1 << 28) // K)), "K": K, "p4": p4, "p6": p6, "p8": p8,
                "fp6": fp6, "fp8": fp8}
    N = _log(rng, 512, 28672)
    M = _log(rng, 1, max(1, min(8192, MAX_MNK // (N * K))))
    return _linear("", M, K, N, (p4, p6, p8), norm=rng.random() < 0.4, kept=rng.random() < 0.5, fp6=fp6, fp8=fp8)


# ---- inputs ----


def _generator(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + k)
    return g


def _activations(seed, k, M, K):
    """bf16 [M, K] with a few large channels, and sigma: the regular channels in a random order, then the large ones."""
    g = _generator(seed, k)
    order = torch.randperm(K, generator=g, device="cuda")
    n = round(OUTLIERS * K)
    x = torch.randn((M, K), generator=g, device="cuda")
    if n:
        x[:, order[K - n:]] *= OUTLIER_SCALE
    return x.to(torch.bfloat16), order.to(torch.int32)


def _weight(seed, k, N, K):
    return torch.randn((N, K), generator=_generator(seed, k), device="cuda").mul_(W_STD).to(torch.bfloat16)


def _gamma(seed, k, K):
    return (1.0 + 0.25 * torch.randn(K, generator=_generator(seed, k), device="cuda")).to(torch.bfloat16)


def _linears(case):
    """The case's linear layers as (M, K, N, split, norm, formats)."""
    if case["op"] == "layer":
        return [(case["M"], K, N, _split(K), norm, B.DEFAULT_FORMATS) for K, N, norm in LAYER]
    return [(case["M"], case["K"], case["N"], (case["p4"], case["p6"], case["p8"]), case["norm"],
             (case["fp6"], case["fp8"]))]


def _linear_inputs(seed, k, lin):
    M, K, N, _, norm, _ = lin
    x, perm = _activations(seed, 10 * k, M, K)
    return x, perm, _gamma(seed, 10 * k + 1, K) if norm else None, _weight(seed, 10 * k + 2, N, K)


def _call(s):
    """One linear layer; `out` and `y` are None where the call makes its own buffers."""
    if s["gamma"] is None:
        q = B.quantize_act(s["x"], s["perm"], s["split"], out=s["out"], formats=s["formats"])
    else:
        q = B.rmsnorm_quantize_act(s["x"], s["gamma"], EPS, s["perm"], s["split"], out=s["out"], formats=s["formats"])
    return q, B.gemm(q, s["w"], y=s["y"])


def _outputs(q, y):
    return {"y": y, **{b: getattr(q, b) for b in ("q4", "q6", "q8", "sc") if getattr(q, b) is not None}}


def prepare(case, seed):
    if case["op"] == "calib":
        g = _generator(seed, 0)
        scale = torch.exp(torch.randn(case["K"], generator=g, device="cuda"))
        x = torch.empty((case["rows"], case["K"]), dtype=torch.bfloat16, device="cuda")
        for r in range(0, case["rows"], 8192):
            x[r:r + 8192] = torch.randn(x[r:r + 8192].shape, generator=g, device="cuda").mul_(scale)
        return {"op": "calib", "x": x, "formats": (case["fp6"], case["fp8"])}
    if case["op"] == "weight":
        _, perm = _activations(seed, 0, 1, case["K"])
        split, formats = (case["p4"], case["p6"], case["p8"]), (case["fp6"], case["fp8"])
        return {"op": "weight", "w": _weight(seed, 1, case["N"], case["K"]), "perm": perm, "split": split,
                "formats": formats, "out": B.MXTensor.empty(case["N"], case["K"], split, formats=formats)}
    kept = case["op"] == "layer" or case["kept"]
    states = []
    for k, lin in enumerate(_linears(case)):
        M, K, N, split, norm, formats = lin
        x, perm, gamma, w = _linear_inputs(seed, k, lin)
        wq = B.quantize_weight(w, perm, split, formats=formats)
        out = B.MXTensor.empty(M, K, split, formats=formats) if kept else None
        y = torch.empty((M, (N + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :N] if kept else None
        states.append({"x": x, "perm": perm, "gamma": gamma, "w": wq, "split": split, "formats": formats, "out": out,
                       "y": y})
    if case["op"] == "linear":
        return {"op": "linear", **states[0]}
    for s in states:  # once before the capture, as any program that captures does
        _call(s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        results = [_call(s) for s in states]
    return {"op": "layer", "graph": graph, "states": states, "outputs": [_outputs(q, y) for q, y in results]}


def run(state):
    if state["op"] == "linear":
        return _outputs(*_call(state))
    if state["op"] == "layer":
        state["graph"].replay()
        return state["outputs"]
    if state["op"] == "weight":
        q = B.quantize_weight(state["w"], state["perm"], state["split"], out=state["out"], formats=state["formats"])
        return {b: getattr(q, b) for b in ("q4", "q6", "q8", "sc") if getattr(q, b) is not None}
    perm, split = B.calibrate(state["x"], formats=state["formats"])
    return {"perm": perm, "split": list(split)}


# ---- what a case cannot do without, and how exact it is ----


def _packed(rows, K, split):
    """Bytes of a quantised operand's codes and scales."""
    return rows * (split[0] // 2 + split[1] * 3 // 4 + split[2] + K // 32)


def work(case):
    if case["op"] == "calib":
        return {"bytes": 2 * case["rows"] * case["K"] + 4 * case["K"] + 12, "flops": 2 * case["rows"] * case["K"]}
    if case["op"] == "weight":
        N, K = case["N"], case["K"]
        return {"bytes": 2 * N * K + 4 * K + _packed(N, K, (case["p4"], case["p6"], case["p8"])), "flops": 2 * N * K}
    total = {"bytes": 0, "flops": 0}
    for M, K, N, split, norm, _ in _linears(case):
        # activation, sigma (and gamma) and packed weight in; packed activation and bf16 result out
        total["bytes"] += 2 * M * K + (6 if norm else 4) * K + _packed(N, K, split) + _packed(M, K, split) + 2 * M * N
        total["flops"] += 2 * M * N * K
    return total


def tolerance(case):
    # whole numbers (codes, scales, sigma, the split) are bit-exact
    if case["op"] in ("weight", "calib"):
        return "exact"
    # bf16 results of fp32 sums: the error against 64 bits is 1.7e-3 (2-norm) and at most half a bf16 step (2^-8 of a
    # value) plus the sums' own; four times that
    return {"rel": 7e-3, "max": 1.6e-2}


FORMATS = {  # mantissa bits, smallest normal exponent, largest value's exponent, largest value
    "E2M1": (1, 0, 2, 6.0), "E3M2": (2, -2, 4, 28.0), "E2M3": (3, 0, 2, 7.5), "E4M3": (3, -6, 8, 448.0),
    "E5M2": (2, -14, 15, 57344.0)}


def _pow2(e):
    """2^e in 64 bits, e whole and within the normal range."""
    return ((e.long() + 1023) << 52).view(torch.float64)


def _mx(x, fmt):
    """x (64 bits, [rows, 32 n]) rounded to MX blocks of 32 elements of format fmt, as values."""
    m, emin, emax, top = FORMATS[fmt]
    b = x.reshape(x.shape[0], -1, 32)
    amax = b.abs().amax(dim=2, keepdim=True)
    e = (torch.frexp(amax).exponent - 1 - emax).clamp(-127, 127)
    e = torch.where(amax == 0, torch.full_like(e, -127), e)
    v = b * _pow2(-e)
    step = (torch.frexp(v).exponent - 1).clamp(min=emin) - m
    q = (torch.round(v * _pow2(-step)) * _pow2(step)).clamp(-top, top)
    return (q * _pow2(e)).reshape(x.shape)


def _mixed(x, perm, split, formats):
    x = x.double()[:, perm.long()]
    p4, p6, _ = split
    parts = [(x[:, :p4], "E2M1"), (x[:, p4:p4 + p6], formats[0]), (x[:, p4 + p6:], formats[1])]
    return torch.cat([_mx(p, f) for p, f in parts if p.shape[1]], dim=1)


def exact(case, seed):
    if case["op"] in ("weight", "calib"):
        return None
    out = []
    for k, lin in enumerate(_linears(case)):
        M, K, N, split, norm, formats = lin
        x, perm, gamma, w = _linear_inputs(seed, k, lin)
        if norm:  # the norm's own roundings are part of its definition
            r = (1.0 / torch.sqrt(x.double().square().mean(dim=1, keepdim=True) + EPS)).float()
            x = (gamma.float() * (x.float() * r).to(torch.bfloat16).float()).to(torch.bfloat16)
        y = _mixed(x, perm, split, formats) @ _mixed(w, perm, split, formats).T
        out.append({"y": y, "q4": None, "q6": None, "q8": None, "sc": None})
    return out if case["op"] == "layer" else out[0]
