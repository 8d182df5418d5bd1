"""The LDS-ordered copy holds its chunks two to a record, whichever panels they belong to: panels of odd and even numbers of chunks,
streams of waves that begin with a record's second chunk, few panels whose chunks are shared, panels of fewer rows than a
request brings, and new values -- element by element against the CPU oracle."""
import numpy as np
import pytest

from paper_2209_06979_amd import binding as mc
from paper_2209_06979_amd import workloads as wl
from gpu_util import run_spmm_oracle

pytestmark = pytest.mark.gpu


def _values(prec, n, V, seed):
    return (wl.uniform_packed_int4((n, V // 2), seed) if prec[:2] == "L4" else wl.uniform_int16((n, V), seed) if prec[:3] == "L16" else
            wl.uniform_int8((n, V), seed))


@pytest.mark.parametrize("merge", [-1, 1])
@pytest.mark.parametrize("prec,V,K,N", [("L8R8", 8, 2600, 48), ("L8R8", 4, 700, 80), ("L8R4", 8, 900, 96), ("L4R4", 8, 3000, 64), ("L4R4", 2, 640, 160),
                                        ("L16R8", 4, 2700, 32), ("L16R4", 8, 800, 64)])
@pytest.mark.parametrize("panels,longest", [(2, 13), (5, 1), (67, 4), (301, 3)])
def test_records_of_two_chunks(panels, longest, prec, V, K, N, merge):
    import torch
    M = panels * V
    c = wl.spmm_case(M, K, N, V, 0.9, prec, 31 * panels + K)
    counts = np.minimum(K, (np.arange(panels) * 29 % (64 * longest)) + 64 * (np.arange(panels) % longest))   # 0 .. 2 * longest chunks
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(M, K, V, counts, 77)
    n = len(c["col_idx"])
    c["values"] = _values(prec, n, V, 78)
    mc.set_thread_options(mc.Options(spmm_slab=1))
    try:
        A = mc.SparseMatrix(M, K, V, c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[prec])
    finally:
        mc.set_thread_options(None)
    if merge == 1 and not A.merge_group:
        pytest.skip("no merged copy of this operand")
    o = mc.Options(spmm_slab=1, spmm_merge=merge)
    assert mc.spmm_form(A, N, prec, o) == "lds" and mc.spmm_on_merged(A, N, prec, o) == (merge == 1)
    B = torch.from_numpy(np.ascontiguousarray(c["B"])).cuda()
    print(f"records {prec} {M}x{K} N={N} V={V} merge={merge} longest={longest}", flush=True)
    assert np.array_equal(mc.spmm(A, B, prec, options=o).cpu().numpy(), run_spmm_oracle(c))
    c["values"] = _values(prec, n, V, 79)
    A.set_values(torch.from_numpy(np.ascontiguousarray(c["values"])).cuda())
    assert np.array_equal(mc.spmm(A, B, prec, options=o).cpu().numpy(), run_spmm_oracle(c))
    A.close()
