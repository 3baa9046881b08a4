"""Performance cases of the library: what its users have it do, through its public entry points.

`listed()` names the cases, `draw()` makes more of the same ranges, `prepare()` builds what a program holds before the
call (inputs, quantised weights, output and scratch buffers), `run()` is one pass, `work()` the bytes and operations the
pass cannot do without, `tolerance()` how far another correct implementation may be off, and `exact()` the result in
64 bits, computed with plain torch and none of the library's code.

Kinds of cases (key "kind"):
  gemm     one product  C = A . dequant(W)                          (fq.gemm)
  layer    the four products of one decoder layer, one after the other (fq.gemm, four times)
  grouped  the expert products of a mixture-of-experts layer        (fq.gemm_grouped)
  w4a8     the integer path: activations quantised per row, then multiplied (fq.quantize_act_i8, fq.gemm_w4a8)
  offline  what is done once per weight matrix: "adaptive" chooses the group size, quantises and reports the error
           (fq.choose_group, fq.quantize, fq.quant_error); "quantize" only quantises with a given group size; "w4a8"
           quantises for the integer path (fq.quantize_w4a8)
Weights are N(0, 0.02) with 0.1 % of the entries x 20, or 0.02 x Student-t(3) with 1 % of the columns x 50 ("tail");
activations are N(0, 1).
"""
import functools
import math

import torch

from paper_2308_09723_amd import fq, workloads

DEV = "cuda"
LAYERS = workloads.OPT175B_LAYERS
MOE = workloads.MOE
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------------------------------------ the cases
def _gemm(name, M, K, N, act, bits, g, scale="f16", weights="outliers"):
    return {"name": name, "kind": "gemm", "M": M, "K": K, "N": N, "act": act, "bits": bits, "g": g, "scale": scale,
            "weights": weights}


def listed():
    qkv, stress = LAYERS["qkv"], workloads.STRESS_LAYER
    return [
        # the smallest call: a toy layer at decode size, where launch latency and the host's share count
        _gemm("tiny_m4_f16_int4", 4, 1024, 1024, "f16", 4, 128),
        # token-by-token generation, one sequence: all four products of a decoder layer (the weight stream)
        {"name": "decode_layer_m1_f16_int4", "kind": "layer", "M": 1, "act": "f16", "bits": 4, "g": 128,
         "scale": "f16", "weights": "outliers"},
        # generation for a small batch with 8-bit codes and bfloat16 activations, heavy-tailed weights
        _gemm("decode_m16_bf16_int8", 16, *stress, "bf16", 8, 128, weights="tail"),
        # generation for a larger batch: between the memory-bound and the compute-bound regime
        _gemm("batch_m32_bf16_int4", 32, *qkv, "bf16", 4, 128),
        # a short prompt or a wide batch, ragged in rows and columns, group 64 (the paper's own kernels' size)
        _gemm("batch_m200_f16_int4_g64", 200, 8192, 28656, "f16", 4, 64),
        # prompt processing: the compute-bound end
        _gemm("prefill_m2048_bf16_int4", 2048, *qkv, "bf16", 4, 128),
        # the expert products of a mixture-of-experts layer for 2048 tokens, skewed routing, first matrix
        {"name": "moe_prefill_f16_int4", "kind": "grouped", "tokens": MOE["tokens"], "top_k": MOE["top_k"],
         "experts": MOE["experts"], "K": MOE["d_model"], "N": MOE["d_ff"], "act": "f16", "bits": 4, "g": 64},
        # the same layer while generating for 48 sequences, second matrix: a few rows per expert
        {"name": "moe_decode_bf16_int4", "kind": "grouped", "tokens": 48, "top_k": MOE["top_k"],
         "experts": MOE["experts"], "K": MOE["d_ff"], "N": MOE["d_model"], "act": "bf16", "bits": 4, "g": 64},
        # the integer path while generating for a small batch
        {"name": "w4a8_decode_m8", "kind": "w4a8", "M": 8, "K": qkv[0], "N": qkv[1], "g": 128, "act": "f16"},
        # the integer path in prompt processing
        {"name": "w4a8_prefill_m2048", "kind": "w4a8", "M": 2048, "K": qkv[0], "N": qkv[1], "g": 128, "act": "bf16"},
        # loading a checkpoint, floating-point path: group size chosen, matrix quantised, error reported
        {"name": "offline_adaptive_int4", "kind": "offline", "op": "adaptive", "K": stress[0], "N": stress[1],
         "bits": 4, "g": 64, "scale": "f16", "weights": "tail"},
        # loading a checkpoint, integer path
        {"name": "offline_w4a8", "kind": "offline", "op": "w4a8", "K": LAYERS["out_proj"][0],
         "N": LAYERS["out_proj"][1], "bits": 4, "g": 128, "scale": "f16", "weights": "outliers"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shape(rng, most):
    """(K, N) with K a multiple of 128 and N one of 16, K * N at most `most`."""
    K = 128 * _log_int(rng, 8, 128)
    N = 16 * _log_int(rng, 64, 3072)
    return K, min(N, most // K // 16 * 16)


def draw(rng):
    """One more case: a product (half of the draws), a grouped product, the integer path or an offline step."""
    kind = rng.choices(["gemm", "grouped", "w4a8", "offline"], [0.5, 0.16, 0.17, 0.17])[0]
    act = rng.choice(["f16", "bf16"])
    scale = "bf16" if act == "bf16" and rng.random() < 0.25 else "f16"
    bits = rng.choices([4, 8, 3], [0.65, 0.2, 0.15])[0]
    weights = rng.choice(["outliers", "tail"])
    flops_most = 2048 * LAYERS["qkv"][0] * LAYERS["qkv"][1]
    if kind == "gemm":
        M = _log_int(rng, 1, 2048)
        K, N = _shape(rng, min(LAYERS["fc1"][0] * LAYERS["fc1"][1], flops_most // M))
        return {"kind": kind, "M": M, "K": K, "N": N, "act": act, "bits": bits, "g": rng.choice([128, 64, 32, 0]),
                "scale": scale, "weights": weights}
    if kind == "w4a8":
        M = _log_int(rng, 1, 2048)
        K, N = _shape(rng, min(LAYERS["fc1"][0] * LAYERS["fc1"][1], flops_most // M))
        return {"kind": kind, "M": M, "K": K, "N": N, "g": rng.choice([128, 64, 32]), "act": act}
    if kind == "grouped":
        experts = _log_int(rng, 8, 64)
        K, N = _shape(rng, MOE["d_model"] * MOE["d_ff"])
        return {"kind": kind, "tokens": _log_int(rng, 8, MOE["tokens"]), "top_k": rng.choice([1, 2]),
                "experts": experts, "K": K, "N": N, "act": act, "bits": rng.choice([4, 4, 8]),
                "g": rng.choice([128, 64])}
    op = rng.choice(["adaptive", "quantize", "w4a8"])
    K, N = _shape(rng, workloads.STRESS_LAYER[0] * workloads.STRESS_LAYER[1])
    if op == "adaptive":
        # the smallest group the heuristic may choose: halvings of K down to 32 times its odd part (64 at least)
        odd = K // 32
        while odd % 2 == 0:
            odd //= 2
        g = max(64, 32 * odd)
    else:
        g = rng.choice([128, 64, 32]) if op == "w4a8" else rng.choice([128, 64, 32, 0])
    return {"kind": "offline", "op": op, "K": K, "N": N, "bits": 4 if op == "w4a8" else bits, "g": g, "scale": rng.choice(["f16", "bf16"]),
            "weights": weights}


ALPHA = 0.9      # threshold of the group-size heuristic


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed, stream):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 1009 + stream)
    return gen


def _weight(K, N, how, seed, stream=0):
    """One weight matrix, binary16 [K, N] on the GPU."""
    gen = _generator(seed, 100 + stream)
    w = torch.randn((K, N), generator=gen, device=DEV)
    if how == "tail":
        chi = torch.zeros((K, N), device=DEV)
        for _ in range(3):
            chi += torch.randn((K, N), generator=gen, device=DEV).square_()
        w.div_(chi.div_(3.0).sqrt_()).mul_(0.02)
        w.mul_(torch.where(torch.rand((N,), generator=gen, device=DEV) < 0.01, 50.0, 1.0))
        return w.clamp_(-65504.0, 65504.0).to(torch.float16)
    out = torch.rand((K, N), generator=gen, device=DEV) < 1e-3
    return w.mul_(torch.where(out, 0.4, 0.02)).to(torch.float16)


def _activations(M, K, act, seed):
    return torch.randn((M, K), generator=_generator(seed, 7), device=DEV).to(DTYPES[act])


@functools.lru_cache(maxsize=64)
def _routing(tokens, experts, top_k, seed):
    """Row offsets per expert: every token goes to top_k different experts, popularity ~ rank^-1.1 (host list)."""
    gen = torch.Generator().manual_seed(int(seed) * 1009 + 5)
    logp = -MOE["zipf_a"] * torch.arange(1, experts + 1, dtype=torch.float64).log()
    gumbel = -torch.rand((tokens, experts), generator=gen, dtype=torch.float64).clamp_(1e-300).log_().neg_().log_()
    rows = torch.bincount((logp + gumbel).topk(top_k, dim=1).indices.reshape(-1), minlength=experts)
    return tuple([0] + rows.cumsum(0).tolist())


def _scale_format(case):
    return fq.FQ_SCALE_BF16 if case["scale"] == "bf16" else fq.FQ_SCALE_F16


def _products(case):
    """[(K, N)] of the products of a gemm or layer case."""
    return list(LAYERS.values()) if case["kind"] == "layer" else [(case["K"], case["N"])]


def _scratch(nbytes):
    return torch.empty(max(16, nbytes), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("gemm", "layer"):
        M, bits, g = case["M"], case["bits"], case["g"]
        state = {"case": case, "products": []}
        for i, (K, N) in enumerate(_products(case)):
            codes, scales = fq.quantize(_weight(K, N, case["weights"], seed, i), bits, g, _scale_format(case))
            state["products"].append({
                "A": _activations(M, K, case["act"], seed * 8 + i), "codes": codes, "scales": scales,
                "C": torch.empty((M, N), dtype=DTYPES[case["act"]], device=DEV),
                "ws": _scratch(fq.gemm_workspace_bytes(M, N, K, bits, g))})
        return state
    if kind == "grouped":
        E, K, N, bits, g = case["experts"], case["K"], case["N"], case["bits"], case["g"]
        offsets = _routing(case["tokens"], E, case["top_k"], seed)
        per = fq.codes_bytes(K, N, bits)
        codes = torch.empty(E * per, dtype=torch.uint8, device=DEV)
        scales = torch.empty((E, K // g, N), dtype=torch.float16, device=DEV)
        for e in range(E):
            c, s = fq.quantize(_weight(K, N, "outliers", seed, e), bits, g)
            codes[e * per:(e + 1) * per] = c
            scales[e] = s
        return {"case": case, "A": _activations(offsets[-1], K, case["act"], seed), "offsets": list(offsets),
                "codes": codes, "scales": scales.reshape(-1),
                "C": torch.empty((offsets[-1], N), dtype=DTYPES[case["act"]], device=DEV)}
    if kind == "w4a8":
        M, K, N, g = case["M"], case["K"], case["N"], case["g"]
        codes, z, t = fq.quantize_w4a8(_weight(K, N, "outliers", seed), g)
        return {"case": case, "A": _activations(M, K, case["act"], seed), "codes": codes, "z": z, "t": t,
                "C": torch.empty((M, N), dtype=DTYPES[case["act"]], device=DEV),
                "ws": _scratch(fq.gemm_w4a8_workspace_bytes(M, N, K, g))}
    return {"case": case, "W": _weight(case["K"], case["N"], case["weights"], seed)}


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("gemm", "layer"):
        return [fq.gemm(p["A"], p["codes"], p["scales"], case["bits"], case["g"], out=p["C"], workspace=p["ws"])
                for p in state["products"]]
    if kind == "grouped":
        return fq.gemm_grouped(state["A"], state["offsets"], state["codes"], state["scales"], case["bits"], case["g"],
                               case["N"], out=state["C"])
    if kind == "w4a8":
        Aq, alpha = fq.quantize_act_i8(state["A"])
        C = fq.gemm_w4a8(Aq, alpha, state["codes"], state["z"], state["t"], case["g"], DTYPES[case["act"]],
                         out=state["C"], workspace=state["ws"])
        return {"C": C, "Aq": Aq, "alpha": alpha}
    W, bits = state["W"], case["bits"]
    if case["op"] == "w4a8":
        codes, z, t = fq.quantize_w4a8(W, case["g"])
        return {"codes": codes, "z": z, "t": t}
    if case["op"] == "quantize":
        codes, scales = fq.quantize(W, bits, case["g"], _scale_format(case))
        return {"codes": codes, "scales": scales}
    g = fq.choose_group(W, 0, case["g"], ALPHA)
    codes, scales = fq.quantize(W, bits, g, _scale_format(case))
    sse, largest = fq.quant_error(W, codes, scales, bits, g)
    return {"group": g, "codes": codes, "scales": scales, "sse": sse, "largest": largest}


# ------------------------------------------------------------------------------------------------ work and tolerance
def _weight_bytes(K, N, bits, g, scale_bytes=2):
    return K * N * bits // 8 + K // (g or K) * N * scale_bytes


def work(case):
    kind = case["kind"]
    if kind in ("gemm", "layer"):
        M = case["M"]
        shapes = _products(case)
        return {"bytes": sum(_weight_bytes(K, N, case["bits"], case["g"]) + 2 * M * (K + N) for K, N in shapes),
                "flops": sum(2 * M * N * K for K, N in shapes)}
    K, N, g = case["K"], case["N"], case["g"]
    if kind == "grouped":
        # the experts that get rows under one routing of these sizes
        offsets = _routing(case["tokens"], case["experts"], case["top_k"], 0)
        hit = sum(b > a for a, b in zip(offsets, offsets[1:]))
        rows = offsets[-1]
        return {"bytes": hit * _weight_bytes(K, N, case["bits"], g) + 2 * rows * (K + N), "flops": 2 * rows * N * K}
    if kind == "w4a8":
        M = case["M"]
        # activations read once as 16-bit values, their int8 form and scales written once
        return {"bytes": _weight_bytes(K, N, 4, g, 1) + 2 * N + M * (3 * K + 4 + 2 * N), "flops": 2 * M * N * K}
    # offline: the weights are read once, codes and scales written once
    return {"bytes": 2 * K * N + _weight_bytes(K, N, case["bits"], g, 1 if case["op"] == "w4a8" else 2), "flops": 0}


def tolerance(case):
    if case["kind"] == "offline":
        # codes, scales and the group size are whole or correctly rounded; the error sum is a binary64 sum whose
        # order is free (measured against another order: below 1e-13)
        return {"rel": 1e-12, "differ": 0.0}
    # Products: one rounding of the result to its 16-bit type, and of the scaled weight where an implementation
    # brings it to 16 bits before multiplying.  Measured against exact(): 2.1e-4 to 2.8e-4 (f16) and 1.7e-3 (bf16).
    return {"rel": 1.2e-3 if case["act"] == "f16" else 7e-3, "differ": 0.0}


# ------------------------------------------------------------------------------------------------ 64-bit results
def _smallest_scale(two_max, levels, dtype):
    """Smallest value s >= 0 of the 16-bit type `dtype` with levels * s >= two_max (binary64 tensor)."""
    s = (two_max / levels).to(dtype)
    up = (s.view(torch.int16) + 1).view(dtype)
    return torch.where(s.double() * levels < two_max, up, s)


def _codes(W, step, qmax):
    """round_half_even(W / step) clamped; 0 where the step is 0."""
    q = torch.where(step == 0, torch.zeros((), dtype=torch.float64, device=DEV), W / step)
    return q.round_().clamp_(-qmax, qmax)


def _quantised(W, bits, g, dtype):
    """(codes, scales [groups, 1, columns]) of binary64 weights [groups, g, columns]."""
    levels = 2 ** bits - 1
    s = _smallest_scale(2 * W.abs().amax(1, keepdim=True), levels, dtype)
    return _codes(W, s.double(), 2 ** (bits - 1) - 1), s


def _column_chunks(N, width=2048):
    return [(a, min(N, a + width)) for a in range(0, N, width)]


def _product64(A, W, bits, g, dtype):
    """A . dequant(quantise(W)) in binary64."""
    K, N = W.shape
    out = torch.empty((A.shape[0], N), dtype=torch.float64, device=DEV)
    A = A.double()
    for a, b in _column_chunks(N):
        w = W[:, a:b].double().reshape(-1, g or K, b - a)
        q, s = _quantised(w, bits, g, dtype)
        out[:, a:b] = A @ (q * s.double()).reshape(K, b - a)
    return out


def _exact_w4a8_weights(W, g):
    """(codes, multipliers, steps) of binary64 weights [K, columns]: codes [groups, g, columns]."""
    K, n = W.shape
    t = _smallest_scale(2 * W.abs().amax(0), 240, torch.float16)
    w = W.reshape(-1, g, n)
    two_max = 2 * w.abs().amax(1)
    z = torch.where(t == 0, torch.ones((), dtype=torch.float64, device=DEV),
                    torch.ceil(two_max / (15 * t.double()))).clamp_(1, 16)
    return _codes(w, (z * t.double()).unsqueeze(1), 7), z, t


def _exact_group(W, g_min):
    """The heuristic of section 3.3: halve while some group's smaller half is below (1 - alpha) of the group."""
    thr = torch.tensor(1.0) - torch.tensor(ALPHA)                       # binary32
    size = W.shape[0]
    while size % 2 == 0 and size // 2 >= g_min:
        half = W.abs().reshape(-1, 2, size // 2, W.shape[1]).amax(2).float()
        if not bool((half.amin(1) < thr.to(DEV) * half.amax(1)).any()):
            break
        size //= 2
    return size


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gemm", "layer"):
        dtype = DTYPES[case["scale"]]
        return [_product64(_activations(case["M"], K, case["act"], seed * 8 + i),
                           _weight(K, N, case["weights"], seed, i), case["bits"], case["g"], dtype)
                for i, (K, N) in enumerate(_products(case))]
    K, N, g = case["K"], case["N"], case["g"]
    if kind == "grouped":
        offsets = _routing(case["tokens"], case["experts"], case["top_k"], seed)
        A = _activations(offsets[-1], K, case["act"], seed)
        out = torch.empty((offsets[-1], N), dtype=torch.float64, device=DEV)
        for e, (a, b) in enumerate(zip(offsets, offsets[1:])):
            if b > a:
                out[a:b] = _product64(A[a:b], _weight(K, N, "outliers", seed, e), case["bits"], g, torch.float16)
        return out
    if kind == "w4a8":
        A = _activations(case["M"], K, case["act"], seed).double()
        largest = A.abs().amax(1)
        alpha = (largest / 127.5).float()
        alpha = torch.where(alpha.double() * 127.5 < largest, (alpha.view(torch.int32) + 1).view(torch.float32), alpha)
        Aq = _codes(A, alpha.double()[:, None], 127)
        W = _weight(K, N, "outliers", seed)
        C = torch.empty((case["M"], N), dtype=torch.float64, device=DEV)
        for a, b in _column_chunks(N):
            q, z, t = _exact_w4a8_weights(W[:, a:b].double(), g)
            C[:, a:b] = (Aq @ (q * z.unsqueeze(1)).reshape(K, b - a)) * alpha.double()[:, None] * t.double()
        return {"C": C, "Aq": Aq.to(torch.int8), "alpha": alpha.double()}
    W = _weight(K, N, case["weights"], seed)
    if case["op"] == "w4a8":
        parts = [_exact_w4a8_weights(W[:, a:b].double(), g)[1:] for a, b in _column_chunks(N)]
        return {"codes": None, "z": torch.cat([p[0] for p in parts], 1).to(torch.uint8),
                "t": torch.cat([p[1] for p in parts]).double()}
    group = _exact_group(W, g) if case["op"] == "adaptive" else (g or K)
    scales, sse, largest = [], 0.0, 0.0
    for a, b in _column_chunks(N):
        w = W[:, a:b].double().reshape(-1, group, b - a)
        q, s = _quantised(w, case["bits"], group, DTYPES[case["scale"]])
        scales.append(s.squeeze(1))
        err = w - q * s.double()
        sse += float(err.square().sum())
        largest = max(largest, float(err.abs().max()))
    scales = torch.cat(scales, 1).double()
    if case["op"] == "quantize":
        return {"codes": None, "scales": scales}
    return {"group": group, "codes": None, "scales": scales, "sse": sse, "largest": largest}
