"""Heads of 48 bytes in pairs at fewer than 4096 (panel, head) units: from 1152 of them on with three chunks a panel and more."""
import numpy as np
import pytest

import host_library as host


@pytest.mark.parametrize("batch,heads,L,n,want", [
    (1, 8, 1160, 150, (2, 1)),        # 1160 units of three chunks
    (1, 8, 1160, 128, (1, 1)),        # ... of two
    (1, 8, 1144, 150, (1, 1)),        # 1144 of three
    (1, 4, 1160, 580, (1, 2)),        # 580 of ten (two waves: four would make more than 2048)
    (2, 8, 2040, 150, (2, 1)),        # 4080 of three
    (2, 8, 2056, 150, (2, 1)),        # 4112 of three, 12336 in all
    (2, 8, 2056, 128, (1, 1)),        # ... of two, 8224
])
def test_pairs(batch, heads, L, n, want):
    mask = host.Mask(L, np.full(L // 8, n))
    assert mask.attention(batch, heads, 48, 8, 8) == [want]
    assert mask.attention(batch, heads, 48, 16, 8) == [want]
    assert mask.attention(batch, heads, 48, 8, 8, token_major=False)[0][0] == 1
    mask.close()
