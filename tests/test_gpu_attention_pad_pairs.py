"""Two heads of less than 64 elements per workgroup, (L, heads, dk) tensors: one, two and four waves per head, launches that take the
form by themselves, against the CPU oracle and against one head per workgroup."""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,L,batch,heads,sparsity", [(0, 1024, 8, 4, 0.9), (0, 1032, 4, 8, 0.4), (5, 200, 1, 2, 0.5), (3, 1032, 1, 2, 0.6), (4, 1536, 1, 4, 0.1)])
@pytest.mark.parametrize("dk,p_bits,qkv_bits", [(16, 8, 8), (32, 8, 8), (32, 16, 8), (48, 8, 8), (48, 16, 8), (32, 8, 4), (32, 16, 4)])
def test_two_short_heads_per_workgroup(dk, p_bits, qkv_bits, mode, L, batch, heads, sparsity):
    import torch
    from paper_2209_06979_amd import binding as mc
    V = 8
    c = wl.attention_case(batch * heads, L, dk, V, sparsity, 5100 + L)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    if qkv_bits == 4:
        q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in (np.clip(t.astype(np.int32) >> 4, -7, 7) for t in (q, k, v)))
    s_p = np.float32(1.0 / oracle.P_CODE_MAX[p_bits])
    rp, ci = c["row_ptr"], c["col_idx"]
    mask = mc.SparseMatrix(L, L, V, rp, ci)

    def dev(t):
        return torch.from_numpy(np.ascontiguousarray(t)).cuda().reshape(batch, heads, L, -1).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    got = {}
    for m in (mode, 2):
        mc.set_attention_mode(m)
        try:
            got[m] = mc.sparse_attention(dev(q), dev(k), dev(v), mask, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits, out_dtype=torch.float32)
        finally:
            mc.set_attention_mode(0)
    mask.close()
    want, _, probs, _ = oracle.attention(q, k, v, rp, ci, V, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits)
    # codes within fp32 rounding of a half-integer may take either value: a step of s_p times the largest V code each; otherwise the
    # integers are exact, converted and scaled (each rounded to fp32, the scale itself too: 4 x 2^-24)
    x = probs / np.float64(s_p)
    near = (np.abs((x - np.floor(x)) - 0.5) < 1e-4 + 1e-5 * x).reshape(batch * heads, -1, V)
    n_near = np.stack([near[:, rp[p]:rp[p + 1]].sum(axis=1) for p in range(L // V)], axis=1).reshape(batch * heads, L, 1)
    tol = np.abs(want) * 2.0 ** -22 + n_near * float(s_p) * float(s_v) * (7 if qkv_bits == 4 else 127)
    for m, O in got.items():
        err = np.abs(O.reshape(batch * heads, L, dk).cpu().numpy().astype(np.float64) - want)
        assert (err <= tol).all(), f"mode {m}: max error {err.max()}, {(err > tol).sum()} elements beyond their bound"
