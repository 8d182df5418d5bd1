"""The fused attention layer's order of (head group, batch item) pairs -- eight at a time, then the rest -- at numbers of
pairs around and between multiples of eight: every item of a batch equals the same item run alone."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
import input_prep as prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("token_major", [False, True])
@pytest.mark.parametrize("B,heads,dk,p_bits", [(1, 1, 64, 8), (7, 1, 64, 16), (4, 2, 64, 16), (3, 3, 48, 8), (17, 1, 64, 8), (5, 4, 64, 16)])
def test_batched_layers_equal_item_by_item(B, heads, dk, p_bits, token_major):
    import torch
    from paper_2209_06979_amd import binding as mc
    L, V = 264, 8
    c = wl.attention_case(B * heads, L, dk, V, 0.7, 4700 + B)
    (q, s_q), (k, s_k), (v, s_v) = (prep.quantize_inputs_int8(c[n]) for n in "qkv")
    s_p = np.float32(1.0 / (127 if p_bits == 8 else 32639))
    mask = mc.SparseMatrix(L, L, V, c["row_ptr"], c["col_idx"])
    print(f"attention pairs B={B} heads={heads} dk={dk} p_bits={p_bits} token_major={token_major}", flush=True)

    def dev(t):
        x = torch.from_numpy(np.ascontiguousarray(t)).cuda().reshape(B, heads, L, -1)
        return x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) if token_major else x
    qd, kd, vd = dev(q), dev(k), dev(v)
    mc.set_attention_mode(3)                                  # the same number of waves per (panel, head) whatever the size
    try:
        O = mc.sparse_attention(qd, kd, vd, mask, s_q, s_k, s_v, s_p, p_bits=p_bits)
        for b in range(B):
            assert torch.equal(O[b], mc.sparse_attention(qd[b], kd[b], vd[b], mask, s_q, s_k, s_v, s_p, p_bits=p_bits)), b
    finally:
        mc.set_attention_mode(0)


@pytest.mark.parametrize("batch", [4, 8])
def test_fewer_pairs_at_a_time(batch):
    """A mask whose column indices do not fit an XCD's L2 beside a pair's rows: fewer pairs are worked on at a time."""
    import torch
    from paper_2209_06979_amd import binding as mc
    L, V, dk = 8192, 8, 64
    rp, ci = wl.vector_sparse_pattern(L, L, V, 0.9, 4790)
    mask = mc.SparseMatrix(L, L, V, rp, ci)
    g = torch.Generator(device="cuda")
    g.manual_seed(4791)
    q, k, v = (torch.randint(-127, 128, (batch, 1, L, dk), generator=g, device="cuda", dtype=torch.int8) for _ in range(3))
    O = mc.sparse_attention(q, k, v, mask, 0.01, 0.01, 0.01, 1 / 127)
    mc.set_attention_mode(2)                                  # the same number of waves per (panel, head), by panel length alone
    try:
        for b in range(batch):
            assert torch.equal(O[b], mc.sparse_attention(q[b], k[b], v[b], mask, 0.01, 0.01, 0.01, 1 / 127)), b
    finally:
        mc.set_attention_mode(0)
    mask.close()
