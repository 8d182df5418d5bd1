"""The SpMM on all columns has one barrier per step that waits for nothing: another wave may read a stage two steps after it was
written because a wave's writes to LDS come before its reads of the same step, which are waited for.  That order is the kernel's
to keep: stated in the source between the two, and found in what the compiler makes of it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2209_06979_amd import build

SRC = os.path.join(build.CSRC, "spmm_dense_kernels.hip")


def test_the_source_keeps_writes_before_reads():
    with open(SRC) as f:
        loop = f.read().split("for (int s0 = 0; s0 < steps")[1].split("// ---- the sums")[0]
    code = [l.split("//")[0].strip() for l in loop.splitlines()]
    code = [l for l in code if l]
    put, fetch = (next(i for i, l in enumerate(code) if l.startswith(f)) for f in ("put(", "fetch("))
    assert code[put + 1:fetch] == ["in_order();"]


def test_compiled_steps_write_before_they_read(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "dense.s"
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
    subprocess.run([hipcc, *flags, "-x", "hip", "--cuda-device-only", "-S", SRC, "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    text, kernels = out.read_text(), 0
    for body in re.findall(r"^_ZN\w*spmm_dense_kernel\w*:[^\n]*\n(.*?)^\.Lfunc_end", text, re.M | re.S):
        # the steps: between two barriers, with matrix instructions
        ops = re.findall(r"^\s+(s_barrier|ds_write|ds_read\w*_tr|v_mfma)", body, re.M)
        steps = [s.split() for s in " ".join(ops).split("s_barrier")]
        steps = [s for s in steps if "v_mfma" in s]
        assert len(steps) in (4, 8)
        for s in steps:
            lds = [o == "ds_write" for o in s if o != "v_mfma"]
            assert any(lds) and lds == sorted(lds, reverse=True)
        kernels += 1
    assert kernels == 24
