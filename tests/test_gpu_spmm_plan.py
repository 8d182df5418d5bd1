"""The gathered SpMM in the tile and waves that it plans and in every pinned pair equals the CPU oracle, and no pinned pair is expected to be
faster -- rows of one piece and of odd lengths, panels without vectors, work items, two planes, many blocks of columns."""
import numpy as np
import pytest

from paper_2209_06979_amd import binding as mc
from paper_2209_06979_amd import workloads as wl
from gpu_util import run_spmm_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,M,K,V,N,longest", [("L8R8", 8, 64, 8, 16, 1), ("L8R8", 1640, 900, 8, 1040, 9), ("L8R8", 5200, 6000, 2, 48, 3),
                                                  ("L8R4", 520, 3000, 4, 96, 40), ("L4R4", 4104, 1500, 8, 288, 12), ("L4R4", 30, 700, 2, 2080, 6),
                                                  ("L16R8", 1204, 2900, 4, 208, 7), ("L12R4", 640, 5300, 8, 160, 60), ("L16R16", 720, 2000, 8, 264, 20)])
@pytest.mark.parametrize("unequal", [False, True])
def test_the_least_expected_time(prec, M, K, V, N, longest, unequal):
    import torch
    panels = M // V
    c = wl.spmm_case(M, K, N, V, 0.9, prec, 5 * M + N)
    most = min(K, 64 * longest)
    counts = np.full(panels, most)
    if unequal:
        counts = np.where(np.arange(panels) % 17 == 3, most, np.arange(panels) * 13 % 90 % (K + 1))     # 0 .. 89, a few of the longest
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(M, K, V, counts, 7)
    n = len(c["col_idx"])
    c["values"] = (wl.uniform_packed_int4((n, V // 2), 8) if prec == "L4R4" else wl.uniform_int16((n, V), 8) if prec[1] == "1" else
                   wl.uniform_int8((n, V), 8))
    A = mc.SparseMatrix(M, K, V, c["row_ptr"], c["col_idx"], c["values"], mc.LHS_BITS[prec])
    B = torch.from_numpy(np.ascontiguousarray(c["B"])).cuda()
    want = run_spmm_oracle(c)
    print(f"plan {prec} {M}x{K} V={V} N={N} longest={longest} unequal={unequal}", flush=True)
    for merge in (-1, 1) if A.merge_group else (-1,):
        plan = mc.Options(spmm_slab=-1, spmm_merge=merge)
        assert mc.spmm_form(A, N, prec, plan) == "gather"
        us = mc.spmm_form_us(A, N, prec, 4, plan)
        for tile in (64, 128, 256):
            for waves in (1, 2, 4, 8):
                pinned = mc.Options(spmm_slab=-1, spmm_merge=merge, spmm_row_tile_bytes=tile, spmm_waves=waves)
                # (a tile of twice the row and more is no choice; 256 bytes of nibbles run as 128)
                if tile == 64 or tile < 2 * N * mc.RHS_BITS[prec] // 8:
                    assert us <= mc.spmm_form_us(A, N, prec, 4, pinned)
                    assert np.array_equal(mc.spmm(A, B, prec, options=pinned).cpu().numpy(), want), (merge, tile, waves)
        assert np.array_equal(mc.spmm(A, B, prec, options=plan).cpu().numpy(), want)
    assert np.array_equal(mc.spmm(A, B, prec).cpu().numpy(), want)
    A.close()
