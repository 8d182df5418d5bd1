"""New values by whole vectors: every width of a vector and every number of vectors behind a merged one, chunks that end inside a
panel, workgroups with less than four chunks, the largest and smallest values."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import torch_dev, run_spmm_oracle

pytestmark = pytest.mark.gpu

KINDS = [(p, V) for p in ("L4R4", "L8R8", "L16R8", "L16R16") for V in (2, 4, 8)]


@pytest.mark.parametrize("counts", [[1], [64, 65], [0, 200, 0, 0, 3, 130, 64, 7, 1]])
@pytest.mark.parametrize("prec,V", KINDS)
def test_values_of_every_width(prec, V, counts):
    import torch
    from paper_2209_06979_amd import binding as mc
    M, K, N = V * len(counts), 256, 64
    c = wl.spmm_case(M, K, N, V, 0.5, prec, 9500 + V)
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(M, K, V, counts, 9501)
    n = len(c["col_idx"])
    rng = np.random.default_rng(9502)
    if prec == "L4R4":
        sets = [rng.integers(-128, 128, (n, V // 2), dtype=np.int8) for _ in range(2)]
    elif prec == "L8R8":
        sets = [rng.integers(-128, 128, (n, V), dtype=np.int8) for _ in range(2)]
    else:                                      # the ends of what splits into two signed bytes, and the carry between them
        sets = [rng.choice(np.array([-32768, -32640, -129, -128, -1, 0, 127, 128, 255, 32511, 32512, 32639], np.int16), (n, V)) for _ in range(2)]
    mc.set_thread_options(mc.Options(spmm_slab=1, spmm_merge=1))
    try:
        A = mc.SparseMatrix(M, K, V, c["row_ptr"], c["col_idx"], sets[0], mc.LHS_BITS[prec])
    finally:
        mc.set_thread_options(None)
    for values in (sets[1], sets[0]):
        want = run_spmm_oracle(dict(c, values=values))
        A.set_values(torch.from_numpy(values).cuda())
        for merge in (-1, 1):
            for slab in (-1, 1):
                out = torch.full((M, N), -7777777, dtype=torch.int32, device="cuda")
                mc.spmm(A, torch_dev(c["B"]), prec, out=out, options=mc.Options(spmm_merge=merge, spmm_slab=slab))
                assert np.array_equal(out.cpu().numpy(), want), (merge, slab)
    A.close()
