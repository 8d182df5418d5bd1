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


@pytest.mark.parametrize("heads,L,three,want", [
    (8, 4088, 26, (2, 1)),            # 4088 units of 2.05 chunks in the mean
    (8, 4104, 26, (2, 1)), (8, 4944, 6, (2, 1)),     # 4104, and 4944 of 2.01: less than 10000 in all
    (8, 4104, 0, (1, 1)),             # two chunks in every panel
    (8, 1144, 26, (1, 1)),            # 1144 units
])
def test_pairs_of_more_than_two_chunks_in_the_mean(heads, L, three, want):
    lengths = np.full(L // 8, 128)
    lengths[:three] = 150
    mask = host.Mask(L, lengths)
    assert mask.attention(1, heads, 48, 8, 8) == [want]
    assert mask.attention(1, heads, 32, 8, 8)[0][0] == 1          # heads of 32 bytes as before
    mask.close()
