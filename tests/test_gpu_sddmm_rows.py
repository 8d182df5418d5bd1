"""SDDMM on staged rows that do not fill their stage: lengths around the edges of the staged kernel's row classes."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import run_sddmm_gpu, run_sddmm_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,signs,prec,row_bytes",
                         [(V, s, p, r) for V, s in ((8, (False, False)), (2, (False, False)), (4, (True, True)), (8, (True, False)), (8, (False, True)))
                          for p in ("L8R8", "L4R4", "L16R16") if p != "L16R16" or s == (False, False)     # (unsigned operands have 4 or 8 bits)
                          for r in (16, 48, 80, 112, 144, 240, 272, 400, 496, 528, 752, 784, 1008, 1040)])
def test_rows_that_do_not_fill_the_stage(prec, row_bytes, V, signs):
    Kd = row_bytes * 8 // {"L8R8": 8, "L4R4": 4, "L16R16": 16}[prec]
    c = wl.sddmm_case(6 * V, 210, Kd, V, 0.5, prec, 9000 + row_bytes + V)
    c["lhs_unsigned"], c["rhs_unsigned"] = signs
    want = run_sddmm_oracle(c)
    for waves in (-1, 1, 4):
        print(f"sddmm {prec} rows of {row_bytes} bytes V={V} unsigned={signs} waves={waves}", flush=True)
        assert np.array_equal(run_sddmm_gpu(c, waves), want)
