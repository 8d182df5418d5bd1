"""The tile and waves that a gathered SpMM is given: the library's host code without a GPU."""
import pytest

from paper_2209_06979_amd import binding as mc
import host_library as host

SHAPES = [(2048, 4096, 8, 0.9), (4096, 2048, 8, 0.95), (1024, 3000, 4, 0.85), (8192, 4096, 2, 0.97), (256, 2304, 8, 0.7), (512, 700, 8, 0.5), (640, 5000, 4, 0.6)]


@pytest.mark.parametrize("prec", ["L8R8", "L8R4", "L4R4"])
@pytest.mark.parametrize("flags", [1, 2, 3])
def test_unsigned_operands_have_one_chunk_in_flight(prec, flags):
    """Their kernel never has two: what is picked for it does not depend on whether others may, nor is it a pair whose tiles do not fit."""
    for M, K, V, empty in SHAPES:
        A = host.Mat(M, K, V, empty, prec)
        for N in (64, 96, 128, 256, 512, 1024):
            got = A.variant(N, flags=flags)
            assert got == A.variant(N, mc.Options(spmm_stages=1), flags=flags), (M, K, N)
            tile = 12 * (got[0] * (2 if prec != "L8R8" else 1) + 4) * 4
            assert got[0] < 256 and got[1] * max(64 * got[0], tile) <= 65536
        A.close()


@pytest.mark.parametrize("prec", ["L8R8", "L4R4", "L16R8", "L16R16"])
def test_a_dense_operand_beyond_32_bit_offsets_has_one_chunk_in_flight(prec):
    """Rows of B 16 MB and more apart: the launch has one chunk in flight, and its tile and waves are those of that kernel."""
    for M, K, V, empty in SHAPES:
        A = host.Mat(M, K, V, empty, prec)
        gather = mc.Options(spmm_slab=-1, spmm_merge=-1)
        one = mc.Options(spmm_slab=-1, spmm_merge=-1, spmm_stages=1)
        far = (1 << 24) * 8 // A.rhs
        for N in (64, 128, 256, 512):
            assert A.run(N, gather, ex=True)[1] == 2 and A.run(N, gather, ex=True, ld=far)[1] == 1
            assert A.variant(N, gather, ld=far) == A.variant(N, one) == A.variant(N, one, ld=far)
        A.close()


def test_a_small_product_of_two_planes():
    """512 x 512, N = 128: 2.53 - 2.57 us in tiles of 64 bytes by two or four waves, 2.92 in tiles of 128 bytes."""
    A = host.Mat(512, 512, 8, 0.8, "L16R8")
    assert A.variant(128) in ((64, 2), (64, 4))
    A.close()


@pytest.mark.parametrize("prec", ["L8R8", "L8R4", "L4R4", "L16R8", "L16R4", "L12R4", "L16R16"])
@pytest.mark.parametrize("merge", [-1, 1])
def test_the_launch_is_the_pair_with_the_least_expected_time(prec, merge):
    for M, K, V, empty in SHAPES:
        A = host.Mat(M, K, V, empty, prec, options=mc.Options(spmm_merge=merge))
        for row_bytes in (16, 64, 208, 512, 1040):
            N = row_bytes * 8 // A.rhs
            us = {}
            for tile in (64, 128, 256):
                for waves in (1, 2, 4, 8):
                    if (tile == 64 or tile < 2 * row_bytes) and not (tile == 256 and A.rhs == 4):  # (256 bytes of nibbles run as 128)
                        us[tile, waves] = A.us(N, mc.Options(spmm_slab=-1, spmm_merge=merge, spmm_row_tile_bytes=tile, spmm_waves=waves))
            assert us[A.variant(N, mc.Options(spmm_slab=-1, spmm_merge=merge))] == min(us.values())
        A.close()
