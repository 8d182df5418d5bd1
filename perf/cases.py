"""The work that users of this library have it do, as cases that can be timed: SpMM, SDDMM and the sparse
attention layer through the public entry points of the Python binding, from the smallest calls to the largest.

A case is a dict of plain values.  `listed` gives the fixed ones, `draw` one more of the same ranges; `prepare` makes
the inputs and the handles a program keeps, `run` is one pass, `work` what a pass cannot do without.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2209_06979_amd import binding as mc

DEV = "cuda"
SUPPORTED_SDDMM = ("L8R8", "L4R4", "L16R16")
OUT_BYTES = {"int32": 4, "fp32": 4, "fp16": 2}
OUT_TYPE = {"fp32": torch.float32, "fp16": torch.float16}


def listed():
    return [
        # the smallest product: a 512-wide layer, one call at a time, where launch and host time count
        dict(name="spmm_512", op="spmm", prec="L8R8", M=512, K=512, N=128, V=8, sparsity=0.8, skew=0.0, out="int32"),
        # the ordinary pruned layer: 4096 x 4096, nine tenths of the vectors zero, a batch of 256 columns
        dict(name="spmm_4096", op="spmm", prec="L8R8", M=4096, K=4096, N=256, V=8, sparsity=0.9, skew=0.0, out="int32"),
        # the dense end: short vectors, half of them kept, where every row of B is used by many panels
        dict(name="spmm_dense_v2", op="spmm", prec="L8R8", M=4096, K=4096, N=512, V=2, sparsity=0.5, skew=0.0, out="int32"),
        # a convolution lowered to a product, 4-bit on both sides: few rows, a long reduction, fp16 result
        dict(name="spmm_conv_int4", op="spmm", prec="L4R4", M=256, K=2304, N=512, V=8, sparsity=0.7, skew=0.0, out="fp16"),
        # the wide half of a feed-forward block over 1024 tokens, dequantised on the way out (the largest product)
        dict(name="spmm_ffn", op="spmm", prec="L8R8", M=16384, K=4096, N=1024, V=8, sparsity=0.9, skew=0.0, out="fp16"),
        # sizes that are round in nothing, panels of log-normal length as magnitude pruning leaves them, 16-bit weights
        dict(name="spmm_ragged_16", op="spmm", prec="L16R8", M=3004, K=2900, N=208, V=4, sparsity=0.85, skew=1.0, out="int32"),
        # sampled product at a 4096 x 4096 mask: scores of one wide head, or a weight gradient kept at the pattern
        dict(name="sddmm_4096", op="sddmm", prec="L8R8", M=4096, K=4096, Kd=256, V=8, sparsity=0.9, skew=0.0),
        # the same with 16-bit operands, odd sizes and a row length that is no power of two
        dict(name="sddmm_ragged_16", op="sddmm", prec="L16R16", M=2000, K=3100, Kd=200, V=4, sparsity=0.9, skew=0.5),
        # one short sequence (not a power of two long): the attention layer where latency is everything
        dict(name="attention_1000", op="attention", batch=1, heads=4, L=1000, dk=64, sparsity=0.8, p_bits=8, qkv_bits=8,
             order="head", quantize=False, out="fp32"),
        # the layer from fp32 projections: scales measured, inputs quantised, then the fused layer on the
        # token-major tensors a QKV projection writes
        dict(name="attention_4096", op="attention", batch=1, heads=8, L=4096, dk=64, sparsity=0.9, p_bits=8, qkv_bits=8,
             order="token", quantize=True, out="fp16"),
        # a batch of long sequences with 16-bit probabilities (the largest layer)
        dict(name="attention_8x8192", op="attention", batch=8, heads=4, L=8192, dk=64, sparsity=0.9, p_bits=16, qkv_bits=8,
             order="token", quantize=False, out="fp32"),
        # one head step by step, for a program that also wants the probabilities: scores, softmax codes,
        # the codes as an operand's values, product with V
        dict(name="steps_2048", op="steps", L=2048, dk=64, sparsity=0.9, out="fp32"),
    ]


# the most work a drawn case may have: that of the largest listed ones
MOST_GATHERED = 16384 // 8 * 410 * 1024          # SpMM, SDDMM: bytes of rows named by stored vectors
MOST_ATTENTION = 8 * 4 * 1024 * 819 * 2 * 64     # attention: the same over K and V rows
MOST_VECTORS = 4096 // 2 * 2048


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the listed ones' ranges."""
    op = rng.choices(("spmm", "sddmm", "attention", "steps"), (5, 2, 4, 1))[0]
    while True:
        if op in ("spmm", "sddmm"):
            V = rng.choice((2, 4, 8, 8))
            case = dict(op=op, prec=rng.choice(tuple(mc.PREC) if op == "spmm" else SUPPORTED_SDDMM),
                        M=max(1, int(_log(rng, 256, 16384) / V)) * V, K=int(_log(rng, 512, 8192)))
            bits = mc.RHS_BITS[case["prec"]]
            piece = 128 // bits                   # elements of a 16-byte piece: what N and Kd are multiples of
            width = max(1, round(_log(rng, 64, 1024 if op == "spmm" else 512) / piece)) * piece
            case.update({"N" if op == "spmm" else "Kd": width}, V=V, sparsity=round(rng.uniform(0.5, 0.98), 3),
                        skew=rng.choice((0.0, 0.0, 0.0, round(rng.uniform(0.2, 1.2), 2))))
            if op == "spmm":
                case["out"] = rng.choice(("int32", "int32", "fp32", "fp16"))
            nvec = sum(panel_lengths(case["M"] // V, case["K"], case["sparsity"], case["skew"]))
            if nvec <= MOST_VECTORS and nvec * width * bits // 8 <= MOST_GATHERED:
                return case
        elif op == "attention":
            qkv_bits = rng.choice((8, 8, 8, 4))
            dk = rng.choice((64, 64, 64, 128, 32, 96, 160) if qkv_bits == 4 else (64, 64, 64, 128, 32, 48, 80, 96, 112, 160))
            case = dict(op=op, batch=rng.choice((1, 1, 2, 8)), heads=rng.choice((1, 2, 3, 4, 8, 12)),
                        L=int(_log(rng, 256, 8192) / 8) * 8, dk=dk, sparsity=round(rng.uniform(0.7, 0.97), 3),
                        p_bits=rng.choice((8, 8, 16)), qkv_bits=qkv_bits, order=rng.choice(("head", "token")),
                        quantize=rng.choice((False, False, True)), out=rng.choice(("fp32", "fp16")))
            rows = case["batch"] * case["heads"] * case["L"] // 8 * stored(case["L"], case["sparsity"])
            if rows * 2 * dk * qkv_bits // 8 <= MOST_ATTENTION:
                return case
        else:
            return dict(op=op, L=int(_log(rng, 512, 4096) / 8) * 8, dk=rng.choice((32, 64, 64, 128, 256)),
                        sparsity=round(rng.uniform(0.7, 0.97), 3), out=rng.choice(("fp32", "fp16")))


# ------------------------------------------------------------------------------ patterns ----
def stored(K, sparsity):
    """Vectors a panel keeps of its K."""
    return max(8, int(math.floor((1.0 - sparsity) * K + 0.5)))


def panel_lengths(P, K, sparsity, skew):
    """Vectors of every panel: all the same, or quantiles of a log-normal distribution with the same mean."""
    keep = stored(K, sparsity)
    if skew <= 0.0:
        return [keep] * P
    dist = NormalDist(0.0, skew)
    x = [math.exp(dist.inv_cdf((i + 0.5) / P)) for i in range(P)]
    scale = keep * P / sum(x)
    return [min(K, max(1, int(v * scale + 0.5))) for v in x]


def _pattern(gen, P, K, lengths, diagonal=0):
    """Interchange arrays of a random pattern; `diagonal` > 0: that many columns at the panel's own place are kept."""
    counts = torch.tensor(lengths, device=DEV)[torch.randperm(P, generator=gen, device=DEV)]
    most = max(lengths)
    cols = []
    step = max(1, (1 << 25) // K)
    for p0 in range(0, P, step):
        n = min(step, P - p0)
        score = torch.rand((n, K), generator=gen, device=DEV)
        if diagonal:
            own = (torch.arange(p0, p0 + n, device=DEV)[:, None] * diagonal + torch.arange(diagonal, device=DEV))
            score.scatter_(1, own, 2.0)
        best = score.topk(most, dim=1).indices
        best = torch.where(torch.arange(most, device=DEV) < counts[p0:p0 + n, None], best, K).sort(dim=1).values
        cols.append(best[best < K].to(torch.int32))
    row_ptr = torch.cat([counts.new_zeros(1), counts.cumsum(0)]).to(torch.int32)
    return row_ptr.cpu().numpy(), torch.cat(cols).cpu().numpy()


def _integers(gen, rows, cols, bits):
    """Uniform integers: int8, packed nibbles (half the columns), or 16 / 12 bits in [-2048, 2047]."""
    if bits == 4:
        return torch.randint(0, 256, (rows, cols // 2), generator=gen, device=DEV, dtype=torch.uint8)
    if bits == 8:
        return torch.randint(-128, 128, (rows, cols), generator=gen, device=DEV, dtype=torch.int8)
    return torch.randint(-2048, 2048, (rows, cols), generator=gen, device=DEV, dtype=torch.int16)


RMS = {4: 4.6, 8: 73.9, 12: 1182.4, 16: 1182.4}


# --------------------------------------------------------------------------------- passes ----
def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    op = case["op"]
    s = dict(case)
    if op in ("spmm", "sddmm"):
        M, K, V, prec = case["M"], case["K"], case["V"], case["prec"]
        row_ptr, col_idx = _pattern(gen, M // V, K, panel_lengths(M // V, K, case["sparsity"], case["skew"]))
        lhs, rhs = mc.LHS_BITS[prec], mc.RHS_BITS[prec]
        if op == "spmm":
            values = _integers(gen, len(col_idx), V, lhs).cpu().numpy()
            s["A"] = mc.SparseMatrix(M, K, V, row_ptr, col_idx, values, lhs)
            s["B"] = _integers(gen, K, case["N"], rhs)
            s["scale"] = 8.0 / (RMS[lhs] * RMS[rhs] * math.sqrt(stored(K, case["sparsity"])))
        else:
            s["mask"] = mc.SparseMatrix(M, K, V, row_ptr, col_idx)
            s["q"], s["k"] = _integers(gen, M, case["Kd"], lhs), _integers(gen, K, case["Kd"], rhs)
        return s
    L, dk = case["L"], case["dk"]
    row_ptr, col_idx = _pattern(gen, L // 8, L, [stored(L, case["sparsity"])] * (L // 8), diagonal=8)
    s["mask"] = mc.SparseMatrix(L, L, 8, row_ptr, col_idx)
    if op == "steps":
        s["P"] = mc.SparseMatrix(L, L, 8, row_ptr, col_idx, np.zeros((len(col_idx), 8), np.int8), 8)
        x = torch.randn((3, L, dk), generator=gen, device=DEV)
    elif case["order"] == "token":
        x = torch.randn((3, case["batch"], L, case["heads"], dk), generator=gen, device=DEV)
    else:
        x = torch.randn((3, case["batch"], case["heads"], L, dk), generator=gen, device=DEV)
    if op == "attention" and case["quantize"]:
        s["x"] = x
        return s
    # inputs that are integers already: quantised with the range that a calibration run found
    qmax = 7.0 if case.get("qkv_bits") == 4 else 127.0
    s["scales"] = [float(t.abs().max()) / qmax for t in x]
    codes = [mc.quantize(t.contiguous(), sc, case.get("qkv_bits", 8)) for t, sc in zip(x, s["scales"])]
    s["qkv"] = codes if op == "steps" else [_heads_first(t, case) for t in codes]
    return s


def _heads_first(t, case):
    """(batch, heads, L, dk) view, whichever order the tensor is stored in; a batch of one has no batch dimension."""
    if case["order"] == "token":
        t = t.permute(0, 2, 1, 3)
    return t[0] if case["batch"] == 1 else t


def run(s):
    op = s["op"]
    if op == "spmm":
        if s["out"] == "int32":
            return mc.spmm(s["A"], s["B"], s["prec"])
        return mc.spmm_dequant(s["A"], s["B"], s["prec"], s["scale"], OUT_TYPE[s["out"]])
    if op == "sddmm":
        return mc.sddmm(s["q"], s["k"], s["mask"], s["prec"])
    if op == "steps":
        (q, k, v), (s_q, s_k, s_v) = s["qkv"], s["scales"]
        scores = mc.sddmm(q, k, s["mask"], "L8R8")
        codes = mc.sparse_softmax(s["mask"], scores, s_q * s_k / math.sqrt(s["dk"]), 127.0)
        s["P"].set_values(codes)
        return codes, mc.spmm_dequant(s["P"], v, "L8R8", s_v / 127.0, OUT_TYPE[s["out"]])
    p_bits, qkv_bits = s["p_bits"], s["qkv_bits"]
    if s["quantize"]:
        x = s["x"]
        top = torch.empty(3, dtype=torch.float32, device=x.device)
        for i in range(3):
            mc.absmax(x[i], out=top[i:i + 1])
        scales = [m / (7.0 if qkv_bits == 4 else 127.0) for m in top.tolist()]
        q, k, v = (_heads_first(mc.quantize(x[i], scales[i], qkv_bits), s) for i in range(3))
    else:
        (q, k, v), scales = s["qkv"], s["scales"]
    return mc.sparse_attention(q, k, v, s["mask"], *scales, 1.0 / (32639.0 if p_bits == 16 else 127.0), p_bits=p_bits,
                               qkv_bits=qkv_bits, out_dtype=OUT_TYPE[s["out"]])


# -------------------------------------------------------------------- what a pass cannot do without ----
def work(case):
    op = case["op"]
    if op in ("spmm", "sddmm"):
        M, K, V, prec = case["M"], case["K"], case["V"], case["prec"]
        P = M // V
        nvec = sum(panel_lengths(P, K, case["sparsity"], case["skew"]))
        lhs, rhs = mc.LHS_BITS[prec], mc.RHS_BITS[prec]
        pattern = 4 * nvec + 4 * (P + 1)
        if op == "spmm":
            N = case["N"]
            return {"bytes": pattern + nvec * V * lhs / 8 + K * N * rhs / 8 + M * N * OUT_BYTES[case["out"]],
                    "flops": 2 * nvec * V * N}
        return {"bytes": pattern + (M + K) * case["Kd"] * lhs / 8 + 4 * nvec * V, "flops": 2 * nvec * V * case["Kd"]}
    L, dk = case["L"], case["dk"]
    nvec = L // 8 * stored(L, case["sparsity"])
    pattern = 4 * nvec + 4 * (L // 8 + 1)
    if op == "steps":                             # the scores stay inside; the codes come out
        return {"bytes": pattern + 3 * L * dk + 8 * nvec + L * dk * OUT_BYTES[case["out"]], "flops": 4 * nvec * 8 * dk}
    rows = case["batch"] * case["heads"] * L
    inputs = 3 * rows * dk * (4 if case["quantize"] else case["qkv_bits"] / 8)
    return {"bytes": pattern + inputs + rows * dk * OUT_BYTES[case["out"]],
            "flops": 4 * case["batch"] * case["heads"] * nvec * 8 * dk}


def tolerance(case):
    op = case["op"]
    if op == "sddmm" or (op == "spmm" and case["out"] == "int32"):
        return "exact"
    if op == "spmm":                              # one rounding of an exact integer times the scale
        return {"rel": 1e-6 if case["out"] == "fp32" else 1e-3}
    # fp32 softmax: a probability within rounding of a half-integer code may take either code, which moves an output
    # by one step of that code (a few in a million of the 8-bit codes; the steps of 16-bit codes are much finer)
    if case.get("p_bits", 8) == 16:
        return {"rel": 1e-3 if case["out"] == "fp16" else 1e-4, "max": 0.02}
    return {"rel": 2e-3, "max": 0.7, "differ": 1e-4}
