"""The SpMM on an operand held with all its columns, forced in every tile shape at the sizes where it can go wrong: one row, one
column and one chunk, blocks of 16 rows and tiles that the matrix does not fill, chunks that the wave groups cannot share
evenly, empty and full panels, padded B and C -- element by element against the CPU oracle, each output type."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import run_spmm_oracle, torch_dev

pytestmark = pytest.mark.gpu

PRECS = ["L8R8", "L8R4", "L4R4", "L16R8", "L16R4", "L12R4"]
# panels, K, rows of B in 16-byte pieces
SIZES = [(1, 1, 1), (3, 63, 2), (9, 64, 4), (37, 65, 5), (33, 257, 9), (70, 700, 8), (150, 1025, 17), (5, 2049, 3)]


def _operand(c, mode=1):
    from paper_2209_06979_amd import binding as mc
    mc.set_spmm_dense(mode)
    try:
        return mc.SparseMatrix(c["M"], c["K"], c["V"], c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[c["prec"]])
    finally:
        mc.set_spmm_dense()


def _spmm(A, c, tile=-1, pad=0, dequant=None):
    """The whole of C, its columns beyond N (`pad` of them) included."""
    import torch
    from paper_2209_06979_amd import binding as mc
    B = torch_dev(c["B"])
    if pad:
        wide = torch.randint(-128, 128, (B.shape[0], B.shape[1] + 64), dtype=torch.int32, device="cuda").to(B.dtype)
        wide[:, :B.shape[1]] = B
        B = wide[:, :B.shape[1]]
    dt = torch.int32 if dequant is None else dequant[1]
    C = torch.full((c["M"], c["N"] + pad), -77, dtype=dt, device="cuda")
    mc.set_spmm_dense(1, tile)
    try:
        form = mc.spmm_form(A, c["N"], c["prec"])
        if dequant is None:
            mc.spmm(A, B, c["prec"], out=C[:, :c["N"]])
        else:
            mc.spmm_dequant(A, B, c["prec"], dequant[0], dt, out=C[:, :c["N"]])
    finally:
        mc.set_spmm_dense()
    torch.cuda.synchronize()
    return C.cpu().numpy(), form


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("V", [2, 4, 8])
@pytest.mark.parametrize("prec", PRECS)
def test_every_tile_shape(prec, V, size):
    import torch
    panels, K, pieces = size
    N = pieces * (32 if prec[-1] == "4" else 16)
    c = wl.spmm_case(panels * V, K, N, V, 0.5, prec, 9700 + K)
    if panels > 30:                                            # panels from empty to full
        counts = np.arange(panels) * 37 % (K + 1)
        counts[0], counts[-1] = 0, K
        c["row_ptr"], c["col_idx"] = wl.ragged_pattern(panels * V, K, V, counts, 9701)
        n = len(c["col_idx"])
        c["values"] = (wl.uniform_packed_int4((n, V // 2), 9702) if prec[:2] == "L4" else
                       wl.uniform_int16((n, V), 9702) if prec[0:3] in ("L16", "L12") else wl.uniform_int8((n, V), 9702))
    want = run_spmm_oracle(c)
    scale = float(np.float32(1e-4))
    f32 = want.astype(np.float32) * np.float32(scale)          # the integer as fp32, times the scale, each rounded once
    A = _operand(c)
    for tile in range(6):
        print(f"dense spmm {prec} V={V} {size} tile={tile}", flush=True)
        pad = 16 * (tile % 2)
        got, form = _spmm(A, c, tile, pad)
        assert form == "dense"
        assert np.array_equal(got[:, :N], want) and (got[:, N:] == -77).all()
        got, _ = _spmm(A, c, tile, pad, (scale, torch.float32))
        assert np.array_equal(got[:, :N], f32)
        got, _ = _spmm(A, c, tile, pad, (scale, torch.float16))
        assert np.array_equal(got[:, :N].copy().view(np.uint16), f32.astype(np.float16).view(np.uint16)) and (got[:, N:] == -77).all()
    A.close()


@pytest.mark.parametrize("prec", ["L8R8", "L4R4", "L16R8"])
def test_new_values_and_stale_copies(prec):
    """Values replaced on the device reach the copy; a softmax that writes the panel format only leaves it unused."""
    from paper_2209_06979_amd import binding as mc
    c = wl.spmm_case(30 * 8, 500, 96, 8, 0.4, prec, 9750)
    A = _operand(c)
    new = np.ascontiguousarray(np.roll(c["values"], 5, axis=0))
    A.set_values(torch_dev(new))
    got, form = _spmm(A, c)
    assert form == "dense" and np.array_equal(got, run_spmm_oracle(dict(c, values=new)))
    if prec == "L8R8":
        S = np.random.default_rng(9751).integers(-3000, 3000, size=A.nvec * 8).astype(np.int32)
        mc.sparse_softmax_to_mat(A, torch_dev(S), 1e-3, 127.0)
        codes = mc.sparse_softmax(A, torch_dev(S.reshape(1, -1)), 1e-3, 127.0).cpu().numpy().reshape(-1, 8)
        got, form = _spmm(A, c)
        assert form != "dense" and np.array_equal(got, run_spmm_oracle(dict(c, values=codes)))
    A.close()


def test_automatic_choice_and_graph():
    """Half empty with V = 2 the form is taken unasked; its launches replay from a graph; a thread that forbids it gets the others."""
    import torch
    from paper_2209_06979_amd import binding as mc
    c = wl.spmm_case(2048, 2048, 512, 2, 0.5, "L8R8", 9760)
    want = run_spmm_oracle(c)
    A, never = _operand(c, 0), _operand(c, -1)
    assert mc.spmm_form(A, 512, "L8R8") == "dense" and mc.spmm_form(never, 512, "L8R8") != "dense"
    B, out = torch_dev(c["B"]), torch.zeros((2048, 512), dtype=torch.int32, device="cuda")
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        mc.spmm(A, B, "L8R8", out=out)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        mc.spmm(A, B, "L8R8", out=out)
    for _ in range(3):
        out.zero_()
        assert np.array_equal(mc.spmm(never, B, "L8R8").cpu().numpy(), want)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
    A.close(), never.close()


def test_new_values_of_an_unasked_copy():
    """Not read yet, the copy is left behind and products take other forms; read by a product in a graph, it follows the values."""
    import torch
    from paper_2209_06979_amd import binding as mc
    c = wl.spmm_case(2048, 2048, 512, 2, 0.5, "L8R8", 9770)
    rolled = [np.ascontiguousarray(np.roll(c["values"], k, axis=0)) for k in (3, 11, 40)]
    B = torch_dev(c["B"])
    A = _operand(c, 0)
    A.set_values(torch_dev(rolled[0]))
    assert mc.spmm_form(A, 512, "L8R8") != "dense"
    assert np.array_equal(mc.spmm(A, B, "L8R8").cpu().numpy(), run_spmm_oracle(dict(c, values=rolled[0])))
    A.close()

    A, out = _operand(c, 0), torch.zeros((2048, 512), dtype=torch.int32, device="cuda")
    stream, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        mc.spmm(A, B, "L8R8", out=out)
    torch.cuda.synchronize()
    assert mc.spmm_form(A, 512, "L8R8") == "dense"
    with torch.cuda.graph(g, stream=stream):
        mc.spmm(A, B, "L8R8", out=out)
    for new in rolled:
        A.set_values(torch_dev(new))
        assert mc.spmm_form(A, 512, "L8R8") == "dense"
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), run_spmm_oracle(dict(c, values=new)))
    A.close()
