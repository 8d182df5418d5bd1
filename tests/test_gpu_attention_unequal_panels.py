"""The layer on masks of unequal panels, one launch for all of them and one per length class, against the CPU oracle and against one head per
workgroup in one launch.  (Which layers are one launch is shown on the host, in test_host_attention_classes.)"""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu
THREE = [(100, 40), (40, 520), (10, 1200)]        # 150 panels of 1, 9 and 19 chunks
LONG = [(300, 40), (40, 520), (12, 2560)]         # 352 of 1, 9 and 40
TWO = [(100, 1), (28, 900)]                       # 128 of 1 and 15


@pytest.mark.parametrize("panels,heads,dk,p_bits,qkv_bits", [
    (THREE, 2, 64, 8, 8), (THREE, 20, 64, 16, 8), (THREE, 21, 64, 8, 8), (THREE, 3, 160, 8, 8), (THREE, 21, 96, 16, 4),
    (LONG, 3, 96, 8, 8), (LONG, 4, 96, 8, 8), (LONG, 4, 48, 16, 8), (TWO, 10, 32, 8, 8), (TWO, 11, 128, 8, 4),
])
@pytest.mark.parametrize("token_major", [True, False])
def test_unequal_panels(panels, heads, dk, p_bits, qkv_bits, token_major):
    import torch
    from paper_2209_06979_amd import binding as mc
    lengths = np.random.default_rng(9850).permutation(np.concatenate([np.full(n, length) for n, length in panels]))
    L = 8 * len(lengths)
    c = wl.attention_case(heads, L, dk, 8, 0.9, 9851 + L + dk)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    if qkv_bits == 4:
        q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in (np.clip(t.astype(np.int32) >> 4, -7, 7) for t in (q, k, v)))
    s_p = np.float32(1.0 / oracle.P_CODE_MAX[p_bits])
    rp, ci = wl.ragged_pattern(L, L, 8, list(lengths), 9852)
    mask = mc.SparseMatrix(L, L, 8, rp, ci)

    def dev(t):
        x = torch.from_numpy(np.ascontiguousarray(t)).cuda()
        return x.permute(1, 0, 2).contiguous().permute(1, 0, 2) if token_major else x
    print(f"unequal panels L={L} heads={heads} dk={dk} p={p_bits} qkv={qkv_bits} token_major={token_major}", flush=True)
    got = {}
    for m in (0, 2):
        mc.set_attention_mode(m)
        try:
            got[m] = mc.sparse_attention(dev(q), dev(k), dev(v), mask, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits, out_dtype=torch.float32)
        finally:
            mc.set_attention_mode(0)
    mask.close()
    want, _, probs, _ = oracle.attention(q, k, v, rp, ci, 8, s_q, s_k, s_v, s_p, p_bits=p_bits, qkv_bits=qkv_bits)
    # codes within fp32 rounding of a half-integer may take either value: a step of s_p times the largest V code each; otherwise the
    # integers are exact, converted and scaled (each rounded to fp32, the scale itself too: 4 x 2^-24)
    x = probs / np.float64(s_p)
    near = (np.abs((x - np.floor(x)) - 0.5) < 1e-4 + 1e-5 * x).reshape(heads, -1, 8)
    n_near = np.stack([near[:, rp[p]:rp[p + 1]].sum(axis=1) for p in range(L // 8)], axis=1).reshape(heads, L, 1)
    tol = np.abs(want) * 2.0 ** -22 + n_near * float(s_p) * float(s_v) * (7 if qkv_bits == 4 else 127)
    for m, O in got.items():
        err = np.abs(O.cpu().numpy().astype(np.float64) - want)
        assert (err <= tol).all(), f"mode {m}: max error {err.max()}, {(err > tol).sum()} elements beyond their bound"
