"""SDDMM on masks whose panels are cut into shares, at the edges of a share (a panel that just needs one more, a last share of one
vector, empty panels, few and many panels), and int16 operands at the ends of their range: element by element against the
oracle, every output type, cut and whole."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


def _case(prec, V, panels, Kd, Nc=1500):
    # 64-vector chunks: panels of 0 .. 23 of them, one vector more or less than whole ones among them
    counts = [(0, 1, 63, 64, 65, 128, 129, 447, 449, 1500, 17, 700)[i % 12] for i in range(panels)]
    c = wl.sddmm_case(panels * V, Nc, Kd, V, 0.5, prec, 9600 + Kd + V)
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(panels * V, Nc, V, counts, 9601)
    if prec == "L16R16":    # the ends of the range against small values: every sum fits 32 bits
        rng = np.random.default_rng(9602)
        ends = np.array([32639, -32768, 127, 128, -128, -129, 255, 256, -1, 0], np.int16)
        c["Kmat"][::2] = rng.choice(ends, c["Kmat"][::2].shape)
        c["Kmat"][1::2] = rng.integers(-60, 61, c["Kmat"][1::2].shape)
        c["Q"] = rng.integers(-60, 61, c["Q"].shape).astype(np.int16)
        c["Q"][::3] = rng.choice(np.array([60, -60, 0], np.int16), c["Q"][::3].shape)
    return c


@pytest.mark.parametrize("panels", [13, 260])
@pytest.mark.parametrize("V", [2, 4, 8])
@pytest.mark.parametrize("prec,Kd", [("L8R8", 48), ("L8R8", 128), ("L8R8", 272), ("L8R8", 400), ("L4R4", 64), ("L4R4", 352), ("L16R16", 24),
                                     ("L16R16", 64), ("L16R16", 200), ("L16R16", 264), ("L16R16", 520)])
def test_cut_masks(prec, Kd, V, panels):
    import torch
    import oracle
    from paper_2209_06979_amd import binding as mc
    c = _case(prec, V, panels, Kd)
    want = oracle.sddmm(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"], c["Q"], c["Kmat"], prec)
    q, k = torch_dev(c["Q"]), torch_dev(c["Kmat"])
    mask = mc.SparseMatrix(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"])
    scale = float(np.float32(1e-4))
    f32 = want.astype(np.float32) * np.float32(scale)
    for splitting in (0, -1):
        o = mc.Options(spmm_splitting=splitting)
        print(f"sddmm shares {prec} Kd={Kd} V={V} panels={panels} splitting={splitting}", flush=True)
        out = torch.full((mask.nvec * V,), -77, dtype=torch.int32, device="cuda")
        mc.sddmm(q, k, mask, prec, out=out, options=o)
        assert np.array_equal(out.cpu().numpy().reshape(want.shape), want)
        mc.set_thread_options(o)                                   # (the calls below take the thread's options)
        try:
            got = mc.sddmm_dequant(q, k, mask, prec, scale, torch.float32).cpu().numpy().reshape(want.shape)
            assert np.array_equal(got, f32)
            got = mc.sddmm_dequant(q, k, mask, prec, scale, torch.float16).cpu().numpy().reshape(want.shape)
            assert np.array_equal(got.view(np.uint16), f32.astype(np.float16).view(np.uint16))
            to = 120.0 / max(1, int(np.abs(want).max()))
            codes = oracle.requantize_scores(want, to, 8).reshape(-1, V)
            P = mc.SparseMatrix(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"], np.full(codes.shape, 77, np.int8), 8)
            mc.sddmm_to_mat(q, k, P, prec, to)
            B = wl.uniform_int8((c["Nc"], 16), 9603)
            got = mc.spmm(P, torch_dev(B), "L8R8").cpu().numpy()
            P.close()
            assert np.array_equal(got, oracle.spmm(c["M"], c["Nc"], V, c["row_ptr"], c["col_idx"], codes, B, "L8R8"))
        finally:
            mc.set_thread_options(None)
    mask.close()
