"""Masks whose panels are all equally long: most kernels compute a panel's first slot, length and first output instead of reading them.  SDDMM
against the oracle in every kernel; the attention layer (the fused kernel; its tile of 192 in automatic mode, which alone takes it) against the same
mask with one vector less in its last panel, whose other rows have to be the same to the last bit."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("prec,Kd,unsigned", [("L8R8", 64, False), ("L8R8", 208, False), ("L8R8", 1040, False), ("L4R4", 64, False), ("L4R4", 64, True),
                                              ("L4R4", 352, False), ("L8R8", 1040, True), ("L16R16", 200, False)])
def test_sddmm(prec, Kd, unsigned, n):
    import torch
    import oracle
    from paper_2209_06979_amd import binding as mc
    for V, panels in ((8, 257), (2, 9)):
        c = wl.sddmm_case(panels * V, 300, Kd, V, 0.5, prec, 9700 + n)
        c["row_ptr"], c["col_idx"] = wl.ragged_pattern(panels * V, 300, V, [n] * panels, 9701)
        print(f"equal panels {prec} Kd={Kd} n={n} V={V} unsigned={unsigned}", flush=True)
        want = oracle.sddmm(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"], c["Q"], c["Kmat"], prec, lhs_unsigned=unsigned, rhs_unsigned=unsigned)
        mask = mc.SparseMatrix(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"])
        out = torch.full((mask.nvec * V,), -77, dtype=torch.int32, device="cuda")
        # (panels of a mask with fewer than 256 would be cut, and a cut one's parts are read)
        mc.sddmm(torch_dev(c["Q"]), torch_dev(c["Kmat"]), mask, prec, out=out, lhs_unsigned=unsigned, rhs_unsigned=unsigned,
                 options=mc.Options(spmm_splitting=-1))
        assert np.array_equal(out.cpu().numpy().reshape(want.shape), want)
        mask.close()


@pytest.mark.parametrize("mode", [2, 3, 4])
@pytest.mark.parametrize("n,heads,dk,p_bits", [(1, 1, 64, 8), (64, 2, 64, 16), (65, 2, 48, 8), (129, 3, 128, 16), (513, 2, 64, 8), (600, 1, 160, 8)])
def test_attention(n, heads, dk, p_bits, mode):
    import torch
    from paper_2209_06979_amd import binding as mc
    L, P = 640, 80
    g = torch.Generator(device="cuda")
    g.manual_seed(9710 + n)
    q, k, v = (torch.randint(-127, 128, (L, heads, dk), generator=g, device="cuda", dtype=torch.int8).permute(1, 0, 2) for _ in range(3))
    print(f"equal panels attention n={n} heads={heads} dk={dk} p_bits={p_bits} mode={mode}", flush=True)
    rp, ci = wl.ragged_pattern(L, L, 8, [n] * P, 9711)
    shorter = np.concatenate([rp[:-1], rp[-1:] - 1]).astype(rp.dtype)
    equal, other = mc.SparseMatrix(L, L, 8, rp, ci), mc.SparseMatrix(L, L, 8, shorter, ci[:-1])
    mode = mode if dk <= 128 else 0
    assert all(mc.attention_form(m, dk, options=mc.Options(attention_mode=mode)) == "fused" for m in (equal, other))
    mc.set_attention_mode(mode)
    try:
        args = (0.02, 0.02, 0.02, 1.0 / (127 if p_bits == 8 else 32639))
        a = mc.sparse_attention(q, k, v, equal, *args, p_bits=p_bits)
        b = mc.sparse_attention(q, k, v, other, *args, p_bits=p_bits)
        assert torch.isfinite(a).all() and float(a.abs().max()) > 0.1
        assert torch.equal(a[:, :L - 8], b[:, :L - 8])
    finally:
        mc.set_attention_mode(0)
    equal.close()
    other.close()
