"""The padding of an operand's LDS-ordered copy against a walk of its records, step by step as the kernel's waves make it."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_06979_amd", "csrc")
PROGRAM = r"""
#include "internal.h"
#include <cstdio>
int main()
{
    for (int ahead = 1; ahead <= RESIDENT_AHEAD; ++ahead)
        for (int n = 0; n <= 100; ++n) {
            int next = 0;                                   // the next record to request; n records are the reader's own
            for (int d = 0; d < ahead; ++d) ++next;         // before the first step
            for (int i = 0; i < n; i += ahead)
                for (int d = 0; d < ahead; ++d) ++next;     // one in every step of a turn, surplus steps too
            if (next != resident_requests(n, ahead) || next - n > RESIDENT_PADDING) return std::printf("ahead %d n %d: %d beyond\n", ahead, n, next - n), 1;
        }
    return 0;
}
"""


def test_requests_beyond_the_last_record_stay_in_the_padding(tmp_path):
    cxx = shutil.which("g++")
    if not cxx or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no host compiler, or no HIP headers")
    (tmp_path / "walk.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}", str(tmp_path / "walk.cpp"), "-o",
                    str(tmp_path / "walk")], check=True)
    done = subprocess.run([str(tmp_path / "walk")], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout
