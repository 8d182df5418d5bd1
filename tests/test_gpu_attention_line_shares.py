"""(L, heads, dk) tensors whose rows cross lines of 128 bytes differently from head to head: fewer pairs at a time than XCDs, and as many,
against the same layer on (heads, L, dk) tensors, to the last bit; strides of a wider tensor and a batch among them."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads,extra", [(1, 8, 0), (1, 12, 0), (2, 3, 1), (1, 5, 3), (8, 8, 0)])
@pytest.mark.parametrize("dk,p_bits,qkv_bits", [(48, 8, 8), (80, 16, 8), (96, 8, 4), (112, 8, 8), (160, 8, 8)])
def test_token_major_equals_head_major(dk, p_bits, qkv_bits, batch, heads, extra):
    import torch
    from paper_2209_06979_amd import binding as mc
    L = 520
    g = torch.Generator(device="cuda")
    g.manual_seed(9800 + dk + heads)
    cols = dk * qkv_bits // 8
    x = torch.randint(-120, 121, (3, batch, heads, L, cols), generator=g, device="cuda", dtype=torch.int8)
    rp, ci = wl.vector_sparse_pattern(L, L, 8, 0.7, 9801)
    mask = mc.SparseMatrix(L, L, 8, rp, ci)
    print(f"line shares dk={dk} p={p_bits} qkv={qkv_bits} batch={batch} heads={heads}+{extra}", flush=True)
    wide = torch.zeros((3, batch, L, heads + extra, cols), device="cuda", dtype=torch.int8)
    wide[:, :, :, :heads] = x.permute(0, 1, 3, 2, 4)
    token = wide[:, :, :, :heads].permute(0, 1, 3, 2, 4)
    mc.set_attention_mode(2)                                  # one head per workgroup, whatever the order
    try:
        args = (mask, 0.02, 0.02, 0.02, 1.0 / (127 if p_bits == 8 else 32639))
        a = mc.sparse_attention(*x, *args, p_bits=p_bits, qkv_bits=qkv_bits)
        b = mc.sparse_attention(*token, *args, p_bits=p_bits, qkv_bits=qkv_bits)
    finally:
        mc.set_attention_mode(0)
    assert float(a.abs().max()) > 0.01 and torch.equal(a, b)
    mask.close()


@pytest.mark.parametrize("batch,heads", [(1, 8), (1, 12), (2, 6), (8, 8), (1, 2)])
@pytest.mark.parametrize("dk,p_bits,qkv_bits", [(48, 8, 8), (48, 16, 8), (16, 8, 8)])
def test_two_heads_per_workgroup_equal_head_major(dk, p_bits, qkv_bits, batch, heads):
    import torch
    from paper_2209_06979_amd import binding as mc
    L = 520
    g = torch.Generator(device="cuda")
    g.manual_seed(9820 + dk + heads)
    x = torch.randint(-120, 121, (3, batch, heads, L, dk * qkv_bits // 8), generator=g, device="cuda", dtype=torch.int8)
    rp, ci = wl.vector_sparse_pattern(L, L, 8, 0.7, 9821)
    mask = mc.SparseMatrix(L, L, 8, rp, ci)
    print(f"line shares of pairs dk={dk} p={p_bits} batch={batch} heads={heads}", flush=True)
    token = x.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4)
    mc.set_attention_mode(5)                                  # two heads per workgroup where tokens hold neighbouring ones
    try:
        args = (mask, 0.02, 0.02, 0.02, 1.0 / (127 if p_bits == 8 else 32639))
        a = mc.sparse_attention(*x, *args, p_bits=p_bits, qkv_bits=qkv_bits)
        b = mc.sparse_attention(*token, *args, p_bits=p_bits, qkv_bits=qkv_bits)
    finally:
        mc.set_attention_mode(0)
    assert float(a.abs().max()) > 0.01 and torch.equal(a, b)
    mask.close()
