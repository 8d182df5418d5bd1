"""The fused attention layer at head dimensions of 144 to 192, batched, with panels of one chunk up to what four waves share:
against the CPU oracle at the first size, and against the layer run as separate kernels (whose fp32 sums are added in another
order, so that a code next to a rounding boundary may move) at all of them."""
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
    assert O.shape == (B, heads, L, dk) and bool(torch.isfinite(O).all())
    d = (O.float() - Op.float()).abs()
    assert float((d > 1e-6).float().mean()) < 0.02 and float(d.max()) < 0.05 * max(1.0, float(Op.float().abs().max()))
    if L == 128:
        r = [t.reshape(B, heads, L, -1)[1] for t in (q, k, v)]
        want = oracle.attention(*r, c["row_ptr"], c["col_idx"], V, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits)[0]
        bad = np.abs(O[1].float().cpu().numpy() - want) > 1e-3 + np.abs(want) * 2.0 ** -10
        assert bad.mean() < 0.02
