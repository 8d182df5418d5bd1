"""Which LDS-ordered copies an operand and its merged copy are given: the library's host code without a GPU."""
import pytest

from paper_2209_06979_amd import binding as mc
import host_library as host

GATHER, MERGED_GATHER = mc.Options(spmm_slab=-1, spmm_merge=-1), mc.Options(spmm_slab=-1, spmm_merge=1)
LDS, MERGED_LDS = mc.Options(spmm_slab=1, spmm_merge=-1), mc.Options(spmm_slab=1, spmm_merge=1)


@pytest.mark.parametrize("M,K,V,empty,prec", [(7232, 522, 8, 0.73, "L4R4"), (14952, 531, 8, 0.6, "L4R4"), (3060, 2891, 4, 0.85, "L8R4"), (2048, 2048, 8, 0.9, "L8R8"),
                                              (16384, 4096, 8, 0.9, "L8R8"), (9608, 4339, 8, 0.68, "L8R8"), (520, 700, 8, 0.9, "L8R8"), (4096, 640, 8, 0.5, "L16R8"),
                                              (4096, 640, 4, 0.5, "L16R8"), (9600, 6400, 8, 0.7, "L4R4"), (6000, 7000, 8, 0.6, "L8R8"), (4800, 5600, 4, 0.7, "L8R8")])
def test_a_resident_form_that_is_worth_a_copy_has_one(M, K, V, empty, prec):
    """One of the two copies is there where one of them is expected to be a twentieth faster than both gathers at some width, none otherwise,
    and a copy that is there is the better one or gains a tenth beside it."""
    bits = mc.LHS_BITS[prec]
    rhs = (4,) if bits == 4 else (8, 4)
    own = host.Mat(M, K, V, empty, prec)
    full = host.Mat(M, K, V, empty, prec, options=mc.Options(spmm_slab=1, spmm_merge=1))
    merged = full.form(128, MERGED_LDS) & 2
    worth, beside, off = [False, False], [False, False], [1.0, 1.0]
    for r in rhs:
        for A in (own, full):
            A.prec = mc.PREC[f"L{bits}R{r}"]
        for row_bytes in (1024, 512, 256, 128):
            N = row_bytes * 8 // r
            us = [full.us(N, LDS), full.us(N, MERGED_LDS) if merged else 1e30]
            gather = min(full.us(N, GATHER), full.us(N, MERGED_GATHER) if merged else 1e30)
            for i in (0, 1):
                worth[i] |= us[i] < 0.95 * gather
                beside[i] |= us[i] < min(0.95 * gather, 0.9 * us[1 - i])
                off[i] *= min(gather, us[i]) / gather
    has = [own.form(128, LDS) == 1, bool(own.form(128, MERGED_GATHER) & 2) and own.form(128, MERGED_LDS) == 3]
    own.close(), full.close()
    assert host.load().host_live() == 0
    assert any(has) == any(worth)
    if all(worth):
        first = int(off[1] <= off[0])
        assert has[first] and has[1 - first] == beside[1 - first]
    else:
        assert has == worth
