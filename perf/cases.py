"""Workloads that the library is timed on: what a program that uses it has it do, through the Python binding.

Kinds of case
  gemm      one planned C = A x B: A in BFP16, B in bf16, bf16 transposed or BFP16, C in bf16 or BFP16
  block     two chained layers with every operand in BFP16: H = X W1 (BFP16 out), Y = H W2 (bf16 out)
  linear    a layer on fp32 activations: quantise X, then Y = X W
  quantize  fp32 -> BFP16
  decode    BFP16 -> bf16

A plan's tile factors are the first of atb.select_tiles' ranking that the storage formats admit.  Sizes come from the
library's own workloads (256^3, 8192^3, the MLP-shaped and the ragged problem, N = 2048 shapes, the skinny problems)
or are the ordinary sizes of a transformer layer.
"""
import math

import torch

import paper_2511_16041_amd as atb

FLOP_CAP = 2.0 * 8192 ** 3          # no drawn case costs more than the largest listed one


def listed():
    return [
        # the smallest call: launch and latency count
        {"name": "gemm_256", "kind": "gemm", "M": 256, "N": 256, "K": 256, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 1.0},
        # the headline problem
        {"name": "gemm_8192", "kind": "gemm", "M": 8192, "N": 8192, "K": 8192, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 1.0},
        # first layer of a transformer MLP over a batch of 8192 tokens
        {"name": "gemm_mlp", "kind": "gemm", "M": 8192, "N": 14336, "K": 4096, "b": "bf16", "c": "bf16", "row_exp": 6, "sigma": 0.02},
        # edge tiles in every dimension
        {"name": "gemm_ragged", "kind": "gemm", "M": 3000, "N": 5000, "K": 4104, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 0.5},
        # a mid-size problem with too few large tiles to fill the chip
        {"name": "gemm_n2048", "kind": "gemm", "M": 1024, "N": 2048, "K": 4096, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 1.0},
        # odd leading dimension of B and C (a vocabulary or class count that nobody padded)
        {"name": "gemm_odd_n", "kind": "gemm", "M": 1500, "N": 3001, "K": 2056, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 0.5},
        # weight of a linear layer as frameworks keep it (N x K)
        {"name": "gemm_bt", "kind": "gemm", "M": 2048, "N": 4096, "K": 4096, "b": "bf16_t", "c": "bf16", "row_exp": 4, "sigma": 0.02},
        # decode step of a small batch, bf16 weights
        {"name": "skinny_bf16", "kind": "gemm", "M": 16, "N": 8192, "K": 8192, "b": "bf16", "c": "bf16", "row_exp": 4, "sigma": 0.02},
        # decode step of a larger batch, weights in BFP16
        {"name": "skinny_bfp16", "kind": "gemm", "M": 64, "N": 14336, "K": 4096, "b": "bfp16", "c": "bf16", "row_exp": 4, "sigma": 0.02},
        # prefill through an MLP with every operand in BFP16
        {"name": "block_bfp16", "kind": "block", "M": 2048, "N": 14336, "K": 4096, "N2": 4096, "row_exp": 4, "sigma": 0.02},
        # a layer on fp32 activations, quantised on the way in
        {"name": "linear_fp32", "kind": "linear", "M": 512, "N": 4096, "K": 4096, "b": "bf16", "row_exp": 4, "sigma": 0.02},
        # a weight matrix expanded back to bf16
        {"name": "decode_8192", "kind": "decode", "M": 8192, "K": 8192, "row_exp": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["gemm", "block", "linear", "quantize", "decode"], [14, 2, 2, 1, 1])[0]
    K = 8 * _log_int(rng, 8, 1024)
    case = {"kind": kind, "K": K, "row_exp": rng.choice([0, 4, 6])}
    if kind in ("quantize", "decode"):
        case["M"] = _log_int(rng, 16, 8192)
        return case
    case["sigma"] = rng.choice([1.0, 0.5, 0.02])
    if kind == "gemm":
        M, N = _log_int(rng, 1, 8192), _log_int(rng, 64, 14336)
        b, c = rng.choice(["bf16", "bf16", "bf16", "bf16_t", "bfp16", "bfp16"]), "bf16"
        if b != "bf16_t" and rng.random() < 0.2:
            c = "bfp16"
        if c == "bfp16":
            N = -(-N // 8) * 8
        elif b == "bf16" and rng.random() < 0.25:
            N |= 1
        elif rng.random() < 0.7:
            N = -(-N // 64) * 64
        case.update(b=b, c=c)
    elif kind == "linear":
        M, N = _log_int(rng, 1, 4096), 2 * _log_int(rng, 64, 4096)
        case["b"] = rng.choice(["bf16", "bfp16"])
    else:
        M, N = _log_int(rng, 1, 4096), 8 * _log_int(rng, 16, 1792)
        case["N2"] = 8 * _log_int(rng, 16, 1024)
    while 2.0 * M * N * (K + case.get("N2", 0)) > FLOP_CAP:
        M = max(1, M // 2)
    case.update(M=M, N=N)
    return case


# ------------------------------------------------------------------ inputs, from the seed alone

def _activations(gen, M, K, row_exp):
    x = torch.randn((M, K), generator=gen, device="cuda")
    if row_exp:
        x *= torch.exp2(torch.randint(-row_exp, row_exp + 1, (M, 1), generator=gen, device="cuda").float())
    return x


def _inputs(case, seed):
    """The fp32 tensors a case starts from: activations, then the weights, as the operand's format lays them out."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, K = case["kind"], case["K"]
    x = _activations(gen, case["M"], K, case["row_exp"])
    if kind in ("quantize", "decode"):
        return x, None, None
    s = case["sigma"]
    by_columns = kind == "block" or case["b"] != "bf16"       # N x K
    w = torch.randn((case["N"], K) if by_columns else (K, case["N"]), generator=gen, device="cuda") * s
    w2 = torch.randn((case["N2"], case["N"]), generator=gen, device="cuda") * s if kind == "block" else None
    return x, w, w2


def _plan(M, N, K, b, c):
    for choice in atb.select_tiles(M, N, K):
        try:
            return atb.Gemm(M, N, K, *choice.tiles(), b_format=b, c_format=c)
        except atb.AtbError:        # this instance does not carry the storage formats
            continue
    raise ValueError("no instance takes these formats")


def _buffer(M, K):
    return torch.zeros(atb.bfp16_bytes(M, K), dtype=torch.uint8, device="cuda")


def _quantized(x):
    return atb.bfp16_quantize(x, out=_buffer(*x.shape))


def _weights(w, b):
    return _quantized(w) if b == "bfp16" else w.bfloat16()


def prepare(case, seed):
    kind, M, K = case["kind"], case["M"], case["K"]
    x, w, w2 = _inputs(case, seed)
    if kind == "quantize":
        return {"kind": kind, "x": x, "out": _buffer(M, K)}
    if kind == "decode":
        return {"kind": kind, "a": _quantized(x), "M": M, "K": K}
    N = case["N"]
    if kind == "block":
        N2 = case["N2"]
        return {"kind": kind, "a": _quantized(x), "w1": _quantized(w), "w2": _quantized(w2),
                "g1": _plan(M, N, K, "bfp16", "bfp16"), "g2": _plan(M, N2, N, "bfp16", "bf16"),
                "h": _buffer(M, N), "y": torch.empty((M, N2), dtype=torch.bfloat16, device="cuda")}
    b, c = case["b"], case.get("c", "bf16")
    out = _buffer(M, N) if c == "bfp16" else torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    state = {"kind": kind, "w": _weights(w, b), "g": _plan(M, N, K, b, c), "out": out}
    if kind == "linear":
        state.update(x=x, a=_buffer(M, K))
    else:
        state["a"] = _quantized(x)
    return state


def run(state):
    kind = state["kind"]
    if kind == "gemm":
        return {"c": state["g"].run(state["a"], state["w"], state["out"])}
    if kind == "linear":
        a = atb.bfp16_quantize(state["x"], out=state["a"])
        return {"a": a, "c": state["g"].run(a, state["w"], state["out"])}
    if kind == "block":
        h = state["g1"].run(state["a"], state["w1"], state["h"])
        return {"h": h, "y": state["g2"].run(h, state["w2"], state["y"])}
    if kind == "quantize":
        return {"a": atb.bfp16_quantize(state["x"], out=state["out"])}
    return {"x": atb.bfp16_decode(state["a"], state["M"], state["K"])}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    kind, M, K = case["kind"], case["M"], case["K"]
    if kind == "quantize":
        return {"bytes": 5.125 * M * K, "flops": 0}
    if kind == "decode":
        return {"bytes": 3.125 * M * K, "flops": 0}
    N = case["N"]
    if kind == "block":
        N2 = case["N2"]
        return {"bytes": 1.125 * (M * K + K * N + 2 * M * N + N * N2) + 2.0 * M * N2, "flops": 2.0 * M * N * (K + N2)}
    b = 1.125 if case["b"] == "bfp16" else 2.0
    c = 1.125 if case.get("c") == "bfp16" else 2.0
    a = 1.125 if kind == "gemm" else 4.0 + 2 * 1.125
    return {"bytes": a * M * K + b * K * N + c * M * N, "flops": 2.0 * M * N * K}


def tolerance(case):
    if case["kind"] in ("quantize", "decode"):
        return "exact"
    # bf16 results: one rounding of the sum.  Measured against 64 bits: 1.55e-3 to 1.84e-3 in the 2-norm, largest single
    # difference 3.9e-3 (half an ulp, 2^-8 of the value).
    # BFP16 results: a sum on a rounding boundary may take the neighbouring code.  Measured against 64 bits: none to
    # 6e-6 of the bytes; small results are allowed two bytes.
    small = 2.5 / (1.125 * case["M"] * case["N"])
    return {"rel": 7e-3, "max": 1.6e-2, "differ": min(0.01, max(3e-5, small))}


# ------------------------------------------------------------------ the same in 64 bits, plain torch

def _pow2(e):
    return ((e.long() + 1023) << 52).view(torch.float64)


def _codes(x):
    """(mantissas, exponents) of the blocks of 8 along the last dimension: E = 127 + floor(log2 max|x|) (the fp32
    exponent field), m = clamp(rne(x 2^(133 - E)), -127, 127)."""
    blocks = x.double().reshape(x.shape[0], -1, 8)
    top = blocks.abs().amax(dim=2)
    e = torch.where(top > 0, torch.frexp(top)[1] + 126, torch.zeros_like(top, dtype=torch.int32)).clamp(0, 254)
    m = torch.round(blocks * _pow2(133 - e).unsqueeze(2)).clamp(-127, 127)
    return m, e


def _rounded(x):
    m, e = _codes(x)
    return (m * _pow2(e - 133).unsqueeze(2)).reshape(x.shape)


def _packed(x):
    """The buffer that holds x in BFP16: [panels of 64][rows][64] mantissas, then [panels][rows][8] exponents."""
    M, K = x.shape
    P = -(-K // 64)
    m, e = _codes(x)
    off = -(-P * M * 64 // 256) * 256
    buf = torch.zeros(-(-(off + P * M * 8) // 256) * 256, dtype=torch.uint8, device=x.device)
    mp = torch.zeros((M, P * 64), dtype=torch.int8, device=x.device)
    mp[:, :K] = m.reshape(M, K).to(torch.int8)
    ep = torch.zeros((M, P * 8), dtype=torch.uint8, device=x.device)
    ep[:, :K // 8] = e.to(torch.uint8)
    buf[:P * M * 64] = mp.view(torch.uint8).reshape(M, P, 64).transpose(0, 1).reshape(-1)
    buf[off:off + P * M * 8] = ep.reshape(M, P, 8).transpose(0, 1).reshape(-1)
    return buf


def exact(case, seed):
    kind = case["kind"]
    x, w, w2 = _inputs(case, seed)
    if kind == "quantize":
        return {"a": _packed(x)}
    if kind == "decode":
        return {"x": _rounded(x)}
    if kind == "block":
        h = _rounded(x) @ _rounded(w).t().contiguous()
        return {"h": _packed(h), "y": _rounded(h) @ _rounded(w2).t().contiguous()}
    if case["b"] == "bfp16":
        w = _rounded(w).t().contiguous()
    elif case["b"] == "bf16_t":
        w = w.bfloat16().double().t().contiguous()
    else:
        w = w.bfloat16().double()
    y = _rounded(x) @ w
    if kind == "linear":
        return {"a": _packed(x), "c": y}
    return {"c": _packed(y) if case.get("c") == "bfp16" else y}
