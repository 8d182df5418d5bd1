"""Probabilities' scales so small that scores far below a row's largest have codes, in every form that a mode pins, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2209_06979_amd import workloads as wl

pytestmark = pytest.mark.gpu


# base-2 exponent of one step of a score, and of the scale: steps beyond 64 apart with codes for one of them, shorter ones with codes down to 2^-100
@pytest.mark.parametrize("step,s_p", [(70.0, 2.0 ** -84), (100.0, 2.0 ** -106), (20.0, 2.0 ** -106), (64.0, 2.0 ** -62)])
@pytest.mark.parametrize("dk,qkv_bits", [(64, 8), (48, 8), (64, 4)])
@pytest.mark.parametrize("mode", [0, 2, 3, 4, 5])
def test_entries_far_below_the_largest(dk, qkv_bits, mode, step, s_p):
    import torch
    from paper_2209_06979_amd import binding as mc
    heads, L = 2, 1040
    c = wl.attention_case(heads, L, dk, 8, 0.3, 6300 + dk)
    g = np.random.default_rng(6301)
    q, k = (g.integers(-1, 2, (heads, L, dk)).astype(np.int8) for _ in range(2))     # scores of a few units, neighbours of the largest among them
    v = g.integers(-7, 8, (heads, L, dk)).astype(np.int8)
    if qkv_bits == 4:
        q, k, v = (((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).astype(np.uint8) for t in (q, k, v))
    s_q = s_k = np.float32(np.sqrt(step * np.log(2.0) * np.sqrt(dk)))
    s_v, s_p = np.float32(1e-3), np.float32(s_p)
    rp, ci = c["row_ptr"], c["col_idx"]
    mask = mc.SparseMatrix(L, L, 8, rp, ci)
    dev = lambda t: torch.from_numpy(np.ascontiguousarray(t)).cuda().permute(1, 0, 2).contiguous().permute(1, 0, 2)
    print(f"small scale of probabilities dk={dk} qkv={qkv_bits} mode={mode} step={step} s_p={s_p}", flush=True)
    mc.set_attention_mode(mode)
    try:
        got = mc.sparse_attention(dev(q), dev(k), dev(v), mask, s_q, s_k, s_v, s_p, p_bits=16, qkv_bits=qkv_bits, out_dtype=torch.float32)
    finally:
        mc.set_attention_mode(0)
    mask.close()
    want, _, probs, codes = oracle.attention(q, k, v, rp, ci, 8, s_q, s_k, s_v, s_p, p_bits=16, qkv_bits=qkv_bits)
    assert (step >= 64.0 and s_p > 1e-20) or ((codes > 0) & (codes < 32639)).any()
    # An exponent of up to 128 carries the roundings of the scale (products of s_q, s_k, 1 / sqrt(dk), log2 e) and of its product with the score, half a unit of 24 bits each, times
    # its size: 6 x 2^-24 x 128 x ln 2 = 3.2e-5 of a probability, and as much of its code; a code within that of a half-integer may be one off, and one
    # of 32639 that is more than one off a half-integer below it
    x = np.minimum(probs / np.float64(s_p), 32640.0)
    slack = 1e-4 + 4e-5 * x
    off = np.where(np.abs((x - np.floor(x)) - 0.5) < slack, 1, 0) + np.floor(slack).astype(np.int64)
    off = off.reshape(heads, -1, 8)
    n_off = np.stack([off[:, rp[p]:rp[p + 1]].sum(axis=1) for p in range(L // 8)], axis=1).reshape(heads, L, 1)
    # otherwise integers, converted and scaled
    tol = np.abs(want) * 2.0 ** -22 + n_off * float(s_p) * float(s_v) * 7
    err = np.abs(got.cpu().numpy().astype(np.float64) - want)
    assert (err <= tol).all(), f"max error {err.max()}, {(err > tol).sum()} elements beyond their bound"
