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
    and of two the given operand's where it gains 15 % over the merged one, the merged one unless nothing is gained beside that."""
    bits = mc.LHS_BITS[prec]
    rhs = (4,) if bits == 4 else (8, 4)
    own = host.Mat(M, K, V, empty, prec)
    full = host.Mat(M, K, V, empty, prec, options=mc.Options(spmm_slab=1, spmm_merge=1))
    merged = full.form(128, MERGED_LDS) & 2
    worth, beside = [False, False], [False, False]
    for r in rhs:
        for A in (own, full):
            A.prec = mc.PREC[f"L{bits}R{r}"]
        for row_bytes in (1024, 512, 256, 128):
            N = row_bytes * 8 // r
            us = [full.us(N, LDS), full.us(N, MERGED_LDS) if merged else 1e30]
            gather = min(full.us(N, GATHER), full.us(N, MERGED_GATHER) if merged else 1e30)
            for i in (0, 1):
                worth[i] |= us[i] < 0.95 * gather
                beside[i] |= us[i] < min(0.95 * gather, (0.85, 0.95)[i] * us[1 - i])
    has = [own.form(128, LDS) == 1, bool(own.form(128, MERGED_GATHER) & 2) and own.form(128, MERGED_LDS) == 3]
    own.close(), full.close()
    assert host.load().host_live() == 0
    assert any(has) == any(worth)
    if all(worth):
        assert has == [beside[0], not beside[0] or beside[1]]
    else:
        assert has == worth


@pytest.mark.parametrize("M,K,V,empty,sigma,prec,N,form", [
    (14816, 1024, 8, 0.801, 0.6, "L8R4", 1440, 3),    # 21.5 us merged, 27.5 as given
    (4240, 3297, 8, 0.673, 0.62, "L8R4", 2048, 3),    # 31.4, 35.4
    (16384, 4096, 8, 0.9, 0.0, "L8R8", 1024, 1),      # 33.3, 30.1
])
def test_the_faster_of_the_resident_forms(M, K, V, empty, sigma, prec, N, form):
    """Operands of panels of 8 rows of which the two forms were measured in turn."""
    A = host.Mat(M, K, V, empty, prec, sigma=sigma)
    assert A.form(N) == form
    A.close()


@pytest.mark.parametrize("prec,V,s", [("L8R8", 8, 0.8), ("L8R8", 4, 0.9), ("L8R4", 8, 0.7), ("L16R8", 4, 0.8)])
def test_the_resident_form_runs_where_it_is_expected_three_percent_faster(prec, V, s):
    given = {"spmm_merge": -1}
    with_copy = mc.Options(spmm_slab=1, **given)
    A = host.Mat(4096, 4096, V, s, prec, options=with_copy)
    seen = set()
    for row_bytes in range(32, 1040, 16):
        N = row_bytes * 8 // A.rhs
        gathered, resident = A.us(N, mc.Options(spmm_slab=-1, **given)), A.us(N, with_copy)
        assert A.form(N, mc.Options(**given)) == int(1.03 * resident < gathered)
        seen.add(1.03 * resident < gathered)
    A.close()
    assert seen == {False, True}
