"""Waves a SIMD holds of SDDMM kernels with float results whose share was read into vector registers once: the compiler's table of the build."""
import os

import pytest

from paper_2209_06979_amd import build

# <bits, pieces of a row, dequantised, unsigned, 32-bit offsets> / <waves, dequantised, unsigned>: with the share in scalar registers
WAVES = {
    "sddmm_nib32_kernel<2, true, true>": 8, "sddmm_nib32_kernel<4, true, true>": 8,
    "sddmm_staged_kernel<4, 4, true, true, false>": 6, "sddmm_staged_kernel<4, 4, true, false, false>": 8,
    "sddmm_staged_kernel<4, 8, true, false, false>": 5, "sddmm_staged_kernel<16, 32, true, false, false>": 5,
    "sddmm_staged_kernel<8, 8, true, false, true>": 6, "sddmm_staged_kernel<8, 16, true, false, true>": 6,
    "sddmm_staged_kernel<8, 64, true, false, true>": 4,
}


def test_waves_of_dequantising_sddmm():
    path = os.path.join(build.PKG, "_build", "kernel_resources.txt")
    if not os.path.exists(path):
        pytest.skip("the library's table of resources is not there (it is written by a build)")
    with open(path) as f:
        rows = [line.split(None, 8) for line in f]
    waves = {r[8].split("(")[0]: int(r[7]) for r in rows if r[0] == "sddmm_kernels.hip"}
    if any(name.startswith("_Z") for name in waves):
        pytest.skip("names were not demangled")
    assert {name: waves[name] for name in WAVES} == WAVES
