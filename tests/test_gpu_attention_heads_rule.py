"""The automatic choice of heads per workgroup and waves per head, on both sides of its lines (units of (panel, head), chunks of a
launch, bytes of a token and of a row; three chunks by four waves), against the CPU oracle and against one head per workgroup.  (That a launch has
the heads and waves that stand beside its sizes is shown on the host, in test_host_attention_rule.)"""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dk,p_bits,qkv_bits,batch,heads,L,sparsity", [
    (64, 16, 8, 1, 4, 2056, 0.6),     # 1028 units of 13 chunks: two heads, two waves each
    (64, 8, 8, 1, 4, 2040, 0.6),      # 1020 units: one head
    (64, 8, 8, 2, 2, 2056, 0.65),     # 1028 units of 12 chunks, 12336 in all: one head
    (128, 8, 4, 2, 2, 2056, 0.6),     # rows of 64 bytes of nibbles: two heads
    (48, 16, 8, 2, 2, 2056, 0.6),     # tokens of 96 bytes: two heads
    (32, 8, 8, 2, 2, 2056, 0.6),      # tokens of 64 bytes: one head
    (32, 16, 8, 1, 4, 2056, 0.6),     # tokens of 128 bytes, two waves each: two heads
    (32, 8, 8, 1, 4, 2056, 0.45),     # 18 chunks, four waves each: one head
    (32, 8, 4, 1, 8, 1040, 0.2),      # nibbles, tokens of 128 bytes, 1040 units of 13 chunks: two heads
    (48, 8, 8, 8, 4, 1032, 0.9),      # 4128 units of 2 chunks, 8256 in all: one head
    (32, 8, 8, 8, 4, 1032, 0.8),      # ... of 4 chunks: two heads
    (64, 8, 8, 1, 4, 520, 0.7), (96, 16, 8, 1, 3, 520, 0.7), (128, 8, 4, 1, 2, 520, 0.7), (160, 8, 8, 1, 2, 520, 0.7),  # 3 chunks, four waves
    (80, 8, 8, 2, 4, 520, 0.7),       # 520 units of 3 chunks: two waves
    (64, 16, 8, 1, 2, 1024, 0.4), (112, 8, 8, 1, 1, 1032, 0.42), (128, 8, 4, 1, 1, 520, 0.38), (32, 16, 4, 1, 3, 520, 0.38),  # eight waves
    (80, 16, 8, 1, 3, 2736, 0.87), (64, 8, 4, 1, 3, 2736, 0.87), (112, 8, 8, 1, 5, 2048, 0.8),  # 1026 and 1280 units of 6 and 7 chunks: two waves
    (64, 8, 8, 1, 2, 1032, 0.42),     # 258 units of 10 chunks: four (panels beyond 8 chunks: at least two)
])
@pytest.mark.parametrize("token_major", [True, False])
def test_automatic_heads_and_waves(dk, p_bits, qkv_bits, batch, heads, L, sparsity, token_major):
    import torch
    from paper_2209_06979_amd import binding as mc
    V = 8
    c = wl.attention_case(batch * heads, L, dk, V, sparsity, 5300 + L + dk)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    if qkv_bits == 4:
        q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in (np.clip(t.astype(np.int32) >> 4, -7, 7) for t in (q, k, v)))
    s_p = np.float32(1.0 / oracle.P_CODE_MAX[p_bits])
    rp, ci = c["row_ptr"], c["col_idx"]
    mask = mc.SparseMatrix(L, L, V, rp, ci)

    def dev(t):
        x = torch.from_numpy(np.ascontiguousarray(t)).cuda().reshape(batch, heads, L, -1)
        return x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) if token_major else x
    got = {}
    for m in (0, 2):
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
