"""The fused attention layer at head dimensions of 144 to 192, batched, with panels of one chunk up to what four waves share,
and the layer run as separate kernels: every element of both against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("token_major,out", [(False, "fp32"), (True, "fp16")])
@pytest.mark.parametrize("p_bits,qkv_bits", [(8, 8), (16, 8), (8, 4), (16, 4)])
@pytest.mark.parametrize("dk,L,sparsity", [(160, 128, 0.6), (192, 640, 0.6), (160, 1032, 0.3), (144, 1536, 0.1), (192, 2048, 0.0)])
def test_head_dimensions_up_to_192(dk, L, sparsity, p_bits, qkv_bits, token_major, out):
    import torch
    from paper_2209_06979_amd import binding as mc
    if qkv_bits == 4 and dk % 32:
        dk = 160
    B, heads, V = 2, 2, 8
    c = wl.attention_case(B * heads, L, dk, V, sparsity, 4900 + L)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    if qkv_bits == 4:
        nib = [np.clip(t.astype(np.int32) >> 4, -7, 7) for t in (q, k, v)]
        q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in nib)
    s_p = np.float32(1.0 / oracle.P_CODE_MAX[p_bits])
    mask = mc.SparseMatrix(L, L, V, c["row_ptr"], c["col_idx"])
    print(f"wide attention dk={dk} L={L} s={sparsity} {p_bits}b-{qkv_bits}b token_major={token_major} {out}", flush=True)

    def dev(t):
        x = torch.from_numpy(np.ascontiguousarray(t)).cuda().reshape(B, heads, L, -1)
        return x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) if token_major else x
    args = (dev(q), dev(k), dev(v), mask, s_q, s_k, s_v, s_p)
    kw = dict(p_bits=p_bits, qkv_bits=qkv_bits, out_dtype=torch.float16 if out == "fp16" else torch.float32)
    O = mc.sparse_attention(*args, **kw)
    mc.set_attention_mode(1)
    try:
        Op = mc.sparse_attention(*args, **kw)
    finally:
        mc.set_attention_mode(0)
    mask.close()
    assert O.shape == (B, heads, L, dk)
    want, _, probs, _ = oracle.attention(q, k, v, c["row_ptr"], c["col_idx"], V, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits)
    # Codes within fp32 rounding of a half-integer may take either value: a step of s_p times the largest V code each.  Otherwise
    # the integers are exact, converted, scaled (each rounded to fp32, the scale itself too: 4 x 2^-24) and, for fp16, rounded once more.
    x = probs / np.float64(s_p)
    near = (np.abs((x - np.floor(x)) - 0.5) < 1e-4 + 1e-5 * x).reshape(B * heads, -1, V)
    rp = c["row_ptr"]
    n_near = np.stack([near[:, rp[p]:rp[p + 1]].sum(axis=1) for p in range(L // V)], axis=1).reshape(B * heads, L, 1)
    tol = np.abs(want) * 2.0 ** -22 + n_near * float(s_p) * float(s_v) * (7 if qkv_bits == 4 else 127)
    if out == "fp16":
        tol += (np.abs(want) + tol) * 2.0 ** -11 + 2.0 ** -25
    for got in (O, Op):
        err = np.abs(got.reshape(B * heads, L, dk).cpu().numpy().astype(np.float64) - want)
        assert (err <= tol).all(), f"max error {err.max()}, {(err > tol).sum()} elements beyond their bound"


@pytest.mark.parametrize("dk,p_bits,qkv_bits", [(160, 8, 8), (160, 16, 8), (192, 16, 4), (144, 16, 8)])
def test_entry_points_agree_and_no_workspace_is_taken(dk, p_bits, qkv_bits):
    """The entry point without a workspace runs the same kernel, code for code, and the other one neither asks for a workspace
    nor, through the binding, allocates one."""
    import torch
    from paper_2209_06979_amd import binding as mc
    heads, L = 3, 1024
    rp, ci = wl.vector_sparse_pattern(L, L, 8, 0.6, 4990, keep_diagonal=True)
    mask = mc.SparseMatrix(L, L, 8, rp, ci)
    g = torch.Generator(device="cuda")
    g.manual_seed(4991)
    q, k, v = (torch.randint(0, 256, (heads, L, dk * qkv_bits // 8), generator=g, device="cuda", dtype=torch.uint8) for _ in range(3))
    if qkv_bits == 8:
        q, k, v = (t.view(torch.int8) for t in (q, k, v))
    s_p = np.float32(1.0 / oracle.P_CODE_MAX[p_bits])
    args = (q, k, v, mask, 0.002, 0.02 if qkv_bits == 8 else 2.0, 0.01, s_p)
    assert mc.attention_form(mask, dk, qkv_bits) == "fused" and mc.attention_form(mask, dk, qkv_bits, mc.Options(attention_mode=1)) == "scores+spmm"
    mc.sparse_attention(*args, p_bits=p_bits, qkv_bits=qkv_bits)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    O = mc.sparse_attention(*args, p_bits=p_bits, qkv_bits=qkv_bits)
    assert mc.attention_workspace_needed(heads, dk, mask, p_bits) > 1 << 20                # (what the pipeline would use)
    assert torch.cuda.max_memory_allocated() - before <= O.numel() * 4 + 4096
    S = torch.full_like(O, float("nan"))
    mc.sparse_attention_static(*args, S, p_bits=p_bits, qkv_bits=qkv_bits)
    assert torch.equal(O, S)
    mask.close()


def test_sharing_of_long_panels_is_the_pipelines():
    """spmm_splitting = 1 on a mask with panels far above the average: the pipeline runs, with its output rows shared."""
    import torch
    from paper_2209_06979_amd import binding as mc
    heads, L, dk = 2, 2048, 160
    counts = np.full(L // 8, 40)
    counts[[3, 77]] = 2000
    rp, ci = wl.ragged_pattern(L, L, 8, counts, 4995)
    mask = mc.SparseMatrix(L, L, 8, rp, ci)
    x = torch.randint(-127, 128, (heads, L, dk), device="cuda", dtype=torch.int8)
    args = (x, x, x, mask, 0.001, 0.02, 0.01, 1 / 127)
    share, piped = mc.Options(spmm_splitting=1), mc.Options(spmm_splitting=1, attention_mode=1)
    assert mc.attention_form(mask, dk, 8) == "fused" and mc.attention_form(mask, dk, 8, share) == "scores+spmm"
    assert torch.equal(mc.sparse_attention(*args, options=share), mc.sparse_attention(*args, options=piped))
    mask.close()
