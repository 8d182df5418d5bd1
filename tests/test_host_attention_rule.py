"""Heads per workgroup and waves per head of the fused layer, on both sides of the rule's lines: the library's host code without a GPU."""
import numpy as np
import pytest

import host_library as host

# dk, p_bits, qkv_bits, batch, heads, L, empty, (heads, waves) token-major, head-major
EQUAL = [
    (64, 16, 8, 1, 4, 2056, 0.6, (2, 2), (1, 2)),     # 1028 units of 13 chunks
    (64, 8, 8, 1, 4, 2040, 0.6, (1, 2), (1, 2)),      # 1020 units
    (64, 8, 8, 2, 2, 2056, 0.65, (1, 2), (1, 2)),     # 1028 units of 12 chunks, 12336 in all
    (128, 8, 4, 2, 2, 2056, 0.6, (2, 2), (1, 2)),     # rows of 64 bytes of nibbles
    (48, 16, 8, 2, 2, 2056, 0.6, (2, 2), (1, 2)),     # tokens of 96 bytes
    (32, 8, 8, 2, 2, 2056, 0.6, (1, 2), (1, 2)),      # tokens of 64 bytes
    (32, 16, 8, 1, 4, 2056, 0.6, (2, 2), (1, 2)),     # tokens of 128 bytes, two waves each
    (32, 8, 8, 1, 4, 2056, 0.45, (1, 4), (1, 4)),     # 18 chunks, four waves each
    (32, 8, 4, 1, 8, 1040, 0.2, (2, 2), (1, 2)),      # nibbles, tokens of 128 bytes, 1040 units of 13 chunks
    (48, 8, 8, 8, 4, 1032, 0.9, (1, 1), (1, 1)),      # 4128 units of 2 chunks, 8256 in all
    (32, 8, 8, 8, 4, 1032, 0.8, (2, 1), (1, 1)),      # ... of 4 chunks
    (64, 8, 8, 1, 4, 520, 0.7, (1, 4), (1, 4)), (160, 8, 8, 1, 2, 520, 0.7, (1, 4), (1, 4)),     # 3 chunks
    (80, 8, 8, 2, 4, 520, 0.7, (1, 2), (1, 2)),       # 520 units of 3 chunks
    (64, 16, 8, 1, 2, 1024, 0.4, (1, 8), (1, 8)), (128, 8, 4, 1, 1, 520, 0.38, (1, 8), (1, 8)),  # 10 chunks; 6 of nibbles
    (80, 16, 8, 1, 3, 2736, 0.87, (1, 2), (1, 2)), (112, 8, 8, 1, 5, 2048, 0.8, (1, 2), (1, 2)),  # 1026 and 1280 units of 6 and 7 chunks
    (64, 8, 8, 1, 2, 1032, 0.42, (1, 4), (1, 4)),     # 258 units of 10 chunks
    # 128 nibbles: pairs by one and two waves, single heads by four (19 chunks, 4800 units); shorter rows in pairs by four, too
    (128, 8, 4, 1, 8, 4800, 0.75, (1, 4), (1, 4)), (128, 16, 4, 1, 8, 4800, 0.75, (1, 4), (1, 4)), (128, 16, 4, 1, 8, 4800, 0.8, (2, 2), (1, 2)),
    (128, 8, 4, 1, 8, 4800, 0.9, (2, 1), (1, 1)), (64, 8, 4, 1, 8, 4800, 0.75, (2, 4), (1, 4)), (96, 8, 4, 1, 8, 4800, 0.75, (1, 4), (1, 4)),
    (48, 8, 8, 1, 8, 4800, 0.75, (2, 4), (1, 4)),
]


@pytest.mark.parametrize("dk,p_bits,qkv_bits,batch,heads,L,empty,token,head", EQUAL)
def test_equal_panels(dk, p_bits, qkv_bits, batch, heads, L, empty, token, head):
    mask = host.Mask(L, np.full(L // 8, round((1 - empty) * L)))
    assert mask.attention(batch, heads, dk, p_bits, qkv_bits) == [token]
    assert mask.attention(batch, heads, dk, p_bits, qkv_bits, token_major=False) == [head]
    mask.close()


# 256 panels, `n` of them of the long kind; (heads, waves) of the short ones' launch and of the long ones'
@pytest.mark.parametrize("short,long,n,batch,heads,dk,qkv_bits,want", [
    (40, 1240, 77, 1, 1, 64, 4, [(1, 1), (1, 8)]),    # 179 panels of one chunk, nibbles: a wave each (eight by the mean of all, 6.7 chunks)
    (40, 1240, 77, 1, 1, 64, 8, [(1, 1), (1, 8)]),
    (150, 1240, 77, 1, 2, 96, 8, [(1, 4), (1, 8)]),   # three chunks
    (500, 2000, 6, 1, 6, 64, 8, [(1, 1), (1, 8)]),    # 1500 units of 8 chunks, 12000 in all
    (520, 2000, 6, 1, 6, 64, 8, [(2, 2), (1, 8)]),    # ... of 9 chunks, 13500 in all
    (40, 1000, 70, 3, 6, 64, 8, [(2, 1), (2, 2)]),    # 1260 units of 16 chunks, 20160 in all: two heads (by the mean of all, 5.1 chunks, one)
])
def test_classes_of_unequal_panels_go_by_their_own_chunks(short, long, n, batch, heads, dk, qkv_bits, want):
    lengths = np.full(256, short)
    lengths[np.arange(n) * 3] = long
    mask = host.Mask(2048, lengths)
    assert mask.attention(batch, heads, dk, qkv_bits=qkv_bits) == want
    mask.close()


# Pairs by several waves with 16-bit codes: down to a scale of the probabilities of 2^-62, where entries 2^-64 of a row's largest have no codes
@pytest.mark.parametrize("dk,p_bits,qkv_bits,s_p,mode,want", [
    (64, 16, 8, 2.0 ** -62, 0, (2, 2)), (64, 16, 8, 2.0 ** -63, 0, (1, 2)), (48, 16, 8, 2.0 ** -63, 0, (1, 2)),
    (64, 16, 8, 2.0 ** -63, 4, (1, 4)), (64, 16, 8, 2.0 ** -62, 4, (2, 4)), (64, 16, 8, 1e-40, 3, (1, 2)),
    (64, 16, 4, 2.0 ** -63, 0, (2, 2)), (64, 8, 8, 2.0 ** -63, 0, (2, 2)),      # the other kernels' exponents have no such bound
])
def test_scales_of_probabilities_that_pairs_by_several_waves_do_not_take(dk, p_bits, qkv_bits, s_p, mode, want):
    mask = host.Mask(2056, np.full(257, 822))         # 1028 units of 13 chunks
    options = host.mc.Options(attention_mode=mode)
    assert mask.attention(1, 4, dk, p_bits, qkv_bits, options=options, s_p=s_p) == [want]
    mask.close()


def test_pairs_by_one_wave_take_any_scale_of_probabilities():
    mask = host.Mask(2056, np.full(257, 500))         # 4112 units of 8 chunks
    assert mask.attention(2, 8, 64, 16, 8, s_p=2.0 ** -63) == [(2, 1)]
    mask.close()
