"""Which kernel the sparse softmax takes: the host's rule, by itself.  Every split holds the panel, and the splits that measured
best stay chosen at the sizes where they did."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2209_06979_amd import build


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("split")
    (d / "s.cpp").write_text('#include "softmax_split.h"\nextern "C" int split(long longest, long units, int variant)\n'
                             "{ SoftmaxSplit s = softmax_split(longest, units, variant); return s.pieces * 16 + s.waves; }\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", f"-I{build.CSRC}", str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    f = ctypes.CDLL(str(d / "s.so")).split
    f.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_int]
    return lambda longest, units, variant=0: divmod(f(longest, units, variant), 16)


def test_every_split_holds_the_panel(split):
    built = {(2, 1), (4, 1), (8, 1), (12, 1), (16, 1), (2, 4), (4, 4), (4, 8), (16, 4)}
    for longest in range(128, 16385, 128):
        for units in (1, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 4096, 4097, 20480, 20481, 10**6):
            for variant in (0, 1):
                pieces, waves = split(longest, units, variant)
                assert (pieces, waves) in built and pieces * waves * 256 >= longest
                assert variant == 0 or waves > 1
            assert split(longest, units, 2) == (0, 0)
    assert split(16384 + 128, 600) == (0, 0)


@pytest.mark.parametrize("longest,units,want", [
    # single waves beat workgroups by 1.06 - 1.25 here
    (3584, 1792, (16, 1)), (3584, 2048, (16, 1)), (3584, 12288, (16, 1)), (3584, 32768, (16, 1)), (4096, 2048, (16, 1)), (4096, 6144, (16, 1)),
    # and lose by 1.05 - 1.38 here
    (3584, 1280, (4, 4)), (4096, 1280, (4, 4)), (4096, 32768, (4, 4)),
    # four waves of 16 pieces beat eight of 4 by 1.03 - 1.06, and lose by as much to 1.1
    (5120, 1024, (16, 4)), (6144, 896, (16, 4)), (5120, 8192, (16, 4)), (4608, 16384, (16, 4)), (5120, 512, (4, 8)), (8192, 1280, (4, 8)), (8192, 1088, (4, 8))])
def test_the_faster_split(split, longest, units, want):
    assert split(longest, units) == want
