"""The gathered SpMM's form with 64-bit offsets into B (rows 16 MB apart, or a B of more than 4 GiB): every precision, tile and number of waves, merged
panels, unsigned operands and work items, element by element against the CPU oracle."""
import numpy as np
import pytest

from paper_2209_06979_amd import binding as mc
from paper_2209_06979_amd import workloads as wl
from gpu_util import run_spmm_oracle

pytestmark = pytest.mark.gpu
K, STRIDE = 70, (1 << 24) + 16                               # rows of B, bytes from one to the next


@pytest.fixture(scope="module")
def far():
    import torch
    yield torch.empty((K, STRIDE), dtype=torch.uint8, device="cuda")
    torch.cuda.empty_cache()


def _case(prec, V, counts, N, K, seed):
    c = wl.spmm_case(V * len(counts), K, N, V, 0.5, prec, seed)
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(V * len(counts), K, V, counts, seed + 1)
    n, bits = len(c["col_idx"]), mc.LHS_BITS[prec]
    c["values"] = (wl.uniform_packed_int4((n, V // 2), seed) if bits == 4 else wl.uniform_int8((n, V), seed) if bits == 8 else
                   wl.uniform_int16((n, V), seed, -2048, 2047))
    return c


def _apart(storage, B):
    """B in rows of the storage's length."""
    import torch
    Bt = torch.from_numpy(np.ascontiguousarray(B))
    view = storage.view(Bt.dtype)[:, :Bt.shape[1]]
    view.copy_(Bt.cuda())
    return view


def _check(A, c, B, options, **signs):
    import torch
    out = torch.full((c["M"], c["N"]), -7777777, dtype=torch.int32, device="cuda")
    got = mc.spmm(A, B, c["prec"], out=out, options=options, **signs).cpu().numpy()
    want = run_spmm_oracle(dict(c, **signs))
    bad = np.argwhere(got != want)
    assert bad.size == 0, f"{len(bad)} mismatches, first at {bad[0]}: got {got[tuple(bad[0])]} want {want[tuple(bad[0])]}"


@pytest.mark.parametrize("V", [2, 4, 8])
@pytest.mark.parametrize("prec", ["L8R8", "L8R4", "L4R4", "L16R8", "L16R4", "L12R4", "L16R16"])
def test_every_variant(far, prec, V):
    N = 320 * 8 // mc.RHS_BITS[prec]                         # rows of 320 bytes
    c = _case(prec, V, [0, 1, 15, 16, 17, 63, 64, 65, 70, 70, 69, 2, 0, 33], N, K, 8100 + V)
    mc.set_thread_options(mc.Options(spmm_merge=1))
    A = mc.SparseMatrix(c["M"], K, V, c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[prec])
    mc.set_thread_options(None)
    B = _apart(far, c["B"])
    for merge in (-1, 1) if A.merge_group else (-1,):
        for tile in (0, 64, 128, 256):
            for waves in (1, 2, 4, 8) if tile else (0,):
                print(f"far rows {prec} V={V} merge={merge} tile={tile} waves={waves}", flush=True)
                _check(A, c, B, mc.Options(spmm_slab=-1, spmm_merge=merge, spmm_row_tile_bytes=tile, spmm_waves=waves))
    A.close()


@pytest.mark.parametrize("signs", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("prec", ["L8R8", "L8R4", "L4R4"])
def test_unsigned(far, prec, signs):
    N = 208 * 8 // mc.RHS_BITS[prec]
    c = _case(prec, 8, [0, 1, 15, 16, 17, 63, 64, 65, 70, 33], N, K, 8200)
    A = mc.SparseMatrix(c["M"], K, 8, c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[prec])
    B = _apart(far, c["B"])
    for tile in (0, 64, 128):
        for waves in (1, 2, 4, 8) if tile else (0,):
            print(f"far rows, unsigned {prec} {signs} tile={tile} waves={waves}", flush=True)
            _check(A, c, B, mc.Options(spmm_row_tile_bytes=tile, spmm_waves=waves), lhs_unsigned=signs[0], rhs_unsigned=signs[1])
    A.close()


@pytest.mark.parametrize("prec", ["L8R8", "L16R4", "L16R16"])
def test_work_items_and_many_chunks(prec):
    """1200 rows 4 MB apart: panels of 18 chunks that are cut into items, and whole."""
    import torch
    rows, V, N = 1200, 8, 96 * 8 // mc.RHS_BITS[prec]
    storage = torch.empty((rows, (1 << 22) + 16), dtype=torch.uint8, device="cuda")
    c = _case(prec, V, [1150] * 3 + [5] * 200 + [64, 65, 300, 0], N, rows, 8300)
    mc.set_thread_options(mc.Options(spmm_slab=-1))
    A = mc.SparseMatrix(c["M"], rows, V, c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[prec])
    mc.set_thread_options(None)
    B = _apart(storage, c["B"])
    for merge in (-1, 1) if A.merge_group else (-1,):
        for splitting in (0, -1):
            for waves in (0, 1, 8):
                print(f"far rows, items {prec} merge={merge} splitting={splitting} waves={waves}", flush=True)
                _check(A, c, B, mc.Options(spmm_slab=-1, spmm_merge=merge, spmm_splitting=splitting, spmm_waves=waves))
    A.close()
    del B, storage
    torch.cuda.empty_cache()
