"""Two heads per workgroup with 4-bit inputs and 16-bit codes, (L, heads, dk) tensors: one, two and four waves per head and a launch that
takes the form by itself, against the CPU oracle and against one head per workgroup."""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,L,batch,heads,sparsity", [(0, 1024, 4, 4, 0.3), (5, 200, 1, 2, 0.5), (5, 520, 1, 2, 0.015), (3, 1032, 1, 2, 0.6), (4, 1536, 1, 4, 0.1)])
@pytest.mark.parametrize("dk", [64, 128])
def test_pairs_of_nibbles(dk, mode, L, batch, heads, sparsity):
    import torch
    from paper_2209_06979_amd import binding as mc
    c = wl.attention_case(batch * heads, L, dk, 8, sparsity, 5200 + L)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in (np.clip(t.astype(np.int32) >> 4, -7, 7) for t in (q, k, v)))
    s_p = np.float32(1.0 / 32639)
    rp, ci = c["row_ptr"], c["col_idx"]
    mask = mc.SparseMatrix(L, L, 8, rp, ci)

    def dev(t):
        return torch.from_numpy(np.ascontiguousarray(t)).cuda().reshape(batch, heads, L, -1).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    want, _, probs, _ = oracle.attention(q, k, v, rp, ci, 8, s_q, s_k, s_v, s_p, p_bits=16, qkv_bits=4)
    # codes within fp32 rounding of a half-integer may take either value: a step of s_p times the largest V code each; otherwise the
    # integers are exact, converted and scaled (each rounded to fp32, the scale itself too: 4 x 2^-24)
    x = probs / np.float64(s_p)
    near = (np.abs((x - np.floor(x)) - 0.5) < 1e-4 + 1e-5 * x).reshape(batch * heads, -1, 8)
    n_near = np.stack([near[:, rp[p]:rp[p + 1]].sum(axis=1) for p in range(L // 8)], axis=1).reshape(batch * heads, L, 1)
    tol = np.abs(want) * 2.0 ** -22 + n_near * float(s_p) * float(s_v) * 7
    for m in (mode, 2):
        print(f"pairs of nibbles dk={dk} L={L} mode={m}", flush=True)
        for out in (torch.float32, torch.float16):
            mc.set_attention_mode(m)
            try:
                got = mc.sparse_attention(dev(q), dev(k), dev(v), mask, s_q, s_k, s_v, s_p, p_bits=16, qkv_bits=4, out_dtype=out)
            finally:
                mc.set_attention_mode(0)
            err = np.abs(got.reshape(batch * heads, L, dk).cpu().numpy().astype(np.float64) - want)
            bound = tol if out == torch.float32 else tol + np.abs(want) * 2.0 ** -11 + 2.0 ** -25
            assert (err <= bound).all(), f"mode {m}: max error {err.max()}, {(err > bound).sum()} elements beyond their bound"
    mask.close()
