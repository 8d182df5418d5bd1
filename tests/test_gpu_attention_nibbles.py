"""Attention on 4-bit Q, K and V at the ends of their range, where scores and sums can be told exactly: scores too small to matter
(every stored entry the same code), and so large that only a row's maxima count."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _packed(x):
    return ((x[..., 0::2] & 15) | ((x[..., 1::2] & 15) << 4)).astype(np.uint8).view(np.int8)


@pytest.mark.parametrize("order", ["head", "token"])
@pytest.mark.parametrize("p_bits", [8, 16])
@pytest.mark.parametrize("dk", [32, 64, 96, 128, 160])
@pytest.mark.parametrize("longest", [200, 900])                 # one wave of a panel's chunks, several
def test_exact_sums_of_extreme_nibbles(longest, dk, p_bits, order):
    import torch
    from paper_2209_06979_amd import binding as mc
    heads, L, V = 2, 1024, 8
    counts = 1 + np.arange(L // V) * 29 % longest
    counts[:3] = longest, 1, 65
    counts[(counts == 2) | (counts == 254)] = 3                 # (127 / n is no half)
    rp, ci = wl.ragged_pattern(L, L, V, counts, 9600)
    rng = np.random.default_rng(9601 + dk)
    q, k, v = (rng.choice(np.array([-8, -8, -7, -1, 0, 1, 6, 7, 7]), (heads, L, dk)).astype(np.int32) for _ in range(3))
    dev = [torch.from_numpy(_packed(x)).cuda() for x in (q, k, v)]
    if order == "token":
        dev = [x.transpose(0, 1).contiguous().transpose(0, 1) for x in dev]
    mask = mc.SparseMatrix(L, L, V, rp, ci)
    pmax = 127 if p_bits == 8 else 32639
    for s in (1e-15, 1e3):
        got = mc.sparse_attention(*dev, mask, s, s, 1.0, 1.0 / pmax, p_bits=p_bits, qkv_bits=4, out_dtype=torch.float32).cpu().numpy().reshape(heads, L, dk)
        for h in range(heads):
            for p in range(L // V):
                c = ci[rp[p]:rp[p + 1]]
                scores = q[h, p * V:(p + 1) * V] @ k[h, c].T
                top = np.ones_like(scores) if s < 1 else (scores == scores.max(axis=1, keepdims=True))
                code = np.rint(pmax / top.sum(axis=1, keepdims=True)) * top
                want = (code @ v[h, c]) / pmax
                # (a code next to a half may fall to either side: 1 of each of them, times 8; and fp32's rounding)
                near = np.abs(pmax / top.sum(axis=1) % 1 - 0.5) < 1e-2
                tol = 1e-6 * np.abs(want) + 1e-6 + np.where(near, 8.0 * top.sum(axis=1) / pmax, 0.0)[:, None]
                assert (np.abs(got[h, p * V:(p + 1) * V] - want) <= tol).all(), (h, p, s)
    mask.close()
