"""The SpMM that keeps a column tile of every row of B in LDS, at the edges of its forms: the numbers of columns where the
tile's width or the number of K-blocks changes, panels from empty to full length, few and many panels per workgroup, the
ragged end of the columns and each output type -- element by element against the CPU oracle."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import run_spmm_oracle
from test_gpu_spmm_slab import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("unequal", [False, True])
@pytest.mark.parametrize("K,prec,V,N", [(7, "L8R8", 8, 16), (2560, "L8R8", 8, 208), (2561, "L16R8", 4, 80), (2560, "L16R4", 8, 96),
                                        (5120, "L4R4", 8, 96), (5121, "L8R8", 4, 144), (5121, "L16R8", 8, 48), (10500, "L8R4", 8, 64)])
@pytest.mark.parametrize("panels", [3, 700])
def test_forms(panels, K, prec, V, N, unequal):
    import torch
    M = panels * V
    c = wl.spmm_case(M, K, N, V, 0.97, prec, 9000 + K)
    if unequal:
        counts = (np.arange(panels) * 37 % 200) * (np.arange(panels) % 5 > 0)
        counts[-1] = K
        c["row_ptr"], c["col_idx"] = wl.ragged_pattern(M, K, V, np.minimum(counts, K), 9001)
        n = len(c["col_idx"])
        c["values"] = (wl.uniform_packed_int4((n, V // 2), 9002) if prec[:2] == "L4" else
                       wl.uniform_int16((n, V), 9002) if prec[:3] == "L16" else wl.uniform_int8((n, V), 9002))
    print(f"resident spmm {prec} {M}x{K} N={N} V={V} unequal={unequal}", flush=True)
    want = run_spmm_oracle(c)
    assert np.array_equal(_run(c), want)
    f32 = want.astype(np.float32) * np.float32(1e-4)           # the integer as fp32, times the scale, each rounded once
    assert np.array_equal(_run(c, dequant=(float(np.float32(1e-4)), torch.float32)), f32)
    f16 = _run(c, dequant=(float(np.float32(1e-4)), torch.float16))
    assert np.array_equal(f16.view(np.uint16), f32.astype(np.float16).view(np.uint16))
