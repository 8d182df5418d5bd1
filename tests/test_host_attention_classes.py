"""Masks of unequal panels: one launch for small layers, one per length class for large ones, on both sides of the lines."""
import numpy as np
import pytest

import host_library as host

THREE = [(100, 40), (40, 520), (10, 1200)]        # 150 panels of 1, 9 and 19 chunks
LONG = [(300, 40), (40, 520), (12, 2560)]         # 352 of 1, 9 and 40
TWO = [(100, 40), (28, 900)]                      # 128 of 1 and 15
APART = [(100, 40), (28, 1020)]                   # 128 of 1 and 16 ...
FAR = [(125, 40), (11, 1080)]                     # 136 of 1 and 17: short and long without a class between


@pytest.mark.parametrize("panels,heads,dk,launches", [
    (THREE, 1, 64, 1), (THREE, 20, 64, 1), (THREE, 21, 64, 3), (THREE, 20, 96, 1), (THREE, 21, 96, 3), (THREE, 20, 160, 1), (THREE, 21, 160, 3),
    (LONG, 3, 96, 1), (LONG, 4, 96, 3), (LONG, 4, 64, 1), (LONG, 8, 64, 1), (LONG, 9, 64, 3), (LONG, 8, 48, 1),
    (TWO, 10, 64, 1), (TWO, 11, 64, 2), (APART, 10, 128, 1), (APART, 11, 128, 2), (FAR, 1, 64, 2),
])
def test_launches(panels, heads, dk, launches):
    lengths = np.concatenate([np.full(n, length) for n, length in panels])
    mask = host.Mask(8 * len(lengths), np.random.default_rng(1).permutation(lengths))
    got = mask.attention(1, heads, dk)
    assert len(got) == launches
    longest = int(lengths.max() + 63) // 64
    assert got[-1][1] >= (8 if longest > 32 else 4 if longest > 16 else 2)       # waves by the longest panel
    mask.close()


def test_pinned_modes_are_one_launch():
    lengths = np.concatenate([np.full(n, length) for n, length in THREE])
    mask = host.Mask(8 * len(lengths), lengths)
    assert [len(mask.attention(1, 40, 64, options=host.mc.Options(attention_mode=m))) for m in (2, 3, 4, 5)] == [1] * 4
    mask.close()
