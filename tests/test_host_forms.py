"""Which form of the SpMM a call takes, by the options and copies it has: the library's host code without a GPU."""
import threading

import pytest

from paper_2209_06979_amd import binding as mc
import host_library as host

# panels whose blocks of 16 rows name every column: the form on the copy with all columns, unasked
DENSE = dict(M=2048, K=2048, V=2, empty=0.5)


@pytest.fixture
def A():
    L = host.load()
    L.mc_set_thread_options(None)
    A = host.Mat(**DENSE)
    yield A
    A.close()
    L.mc_set_thread_options(None)
    assert L.host_live() == 0


def test_thread_choice_of_the_copy_with_all_columns_is_an_option(A):
    """It is seen, set and reset with the thread's other options, and calls with options of their own do not follow it."""
    L = host.load()
    o = mc.Options()
    for mode, tile, want in ((1, -1, 16), (1, 0, 17), (1, 5, 22), (-1, -1, -16), (0, -1, 0)):
        assert L.mc_set_spmm_dense(mode, tile) == 0
        assert L.mc_get_thread_options(o) == 0 and o.spmm_merge == want
    for mode, tile in ((2, -1), (-2, -1), (1, 6), (1, -2)):
        assert L.mc_set_spmm_dense(mode, tile) == mc.MC_EINVAL
    assert A.run(512)[0] == "dense" and A.form(512) == 6
    L.mc_set_spmm_dense(-1, -1)
    assert A.run(512)[0] != "dense" and A.form(512) < 4
    assert A.run(512, ex=True)[0] == "dense" and A.run(512, mc.Options(), ex=True)[0] == "dense" and A.form(512, mc.Options()) == 6
    L.mc_set_spmm_dense(1, 4)
    assert A.run(512) == ("dense", 4)
    assert A.run(512, ex=True) != ("dense", 4)                        # (the automatic tile is another one here)
    assert L.mc_set_thread_options(None) == 0
    assert A.run(512) == A.run(512, ex=True) != ("dense", 4)


def test_every_value_of_the_option(A):
    for tile in range(6):
        assert A.run(512, mc.Options(spmm_merge=mc.SPMM_DENSE + 1 + tile), ex=True) == ("dense", tile)
    assert A.run(512, mc.Options(spmm_merge=mc.SPMM_DENSE), ex=True)[0] == "dense"
    assert A.form(512, mc.Options(spmm_merge=-mc.SPMM_DENSE)) < 4
    assert A.form(512, mc.Options(spmm_merge=1)) in (2, 3) and A.form(512, mc.Options(spmm_merge=-1)) in (0, 1)
    for bad in (-17, -15, -2, 2, 15, 23):
        assert A.form(512, mc.Options(spmm_merge=bad)) == mc.MC_EINVAL
    never = host.Mat(**DENSE, options=mc.Options(spmm_merge=-mc.SPMM_DENSE))
    assert never.form(512) in (0, 1, 2, 3) and never.form(512, mc.Options(spmm_merge=mc.SPMM_DENSE)) < 4
    assert never.form(512, mc.Options(spmm_merge=1)) & 2              # (the merged copy is there)
    never.close()
    small = host.Mat(64, 64, 8, 0.5, options=mc.Options(spmm_merge=mc.SPMM_DENSE))
    assert small.form(64, mc.Options(spmm_merge=mc.SPMM_DENSE)) & 4   # built whatever the shape
    small.close()


def test_a_setter_leaves_the_pin_of_another_copy(A):
    L = host.load()
    o = mc.Options()
    for pin in (1, -1):
        for mode in (-1, 0):
            L.mc_set_thread_options(mc.Options(spmm_merge=pin))
            assert L.mc_set_spmm_dense(mode, -1) == 0
            L.mc_get_thread_options(o)
            assert o.spmm_merge == pin


def test_another_thread_is_not_affected(A):
    L = host.load()
    L.mc_set_spmm_dense(-1, -1)
    seen = []
    t = threading.Thread(target=lambda: seen.append(A.run(512)[0]))
    t.start()
    t.join()
    assert seen == ["dense"] and A.run(512)[0] != "dense"


def test_form_without_options_follows_no_other_default_of_the_thread(A):
    """mc_spmm_form with no options is about mc_spmm_ex with none; of the thread's defaults it knows the copy with all columns only."""
    L = host.load()
    want = [A.form(N, mc.Options()) for N in (16, 64, 512)]
    for o in (mc.Options(spmm_merge=-1), mc.Options(spmm_merge=1), mc.Options(spmm_slab=-1), mc.Options(spmm_waves=2)):
        assert L.mc_set_thread_options(o) == 0
        assert [A.form(N) for N in (16, 64, 512)] == want
    L.mc_set_thread_options(mc.Options(spmm_merge=-mc.SPMM_DENSE, spmm_slab=-1))
    assert [A.form(N) for N in (16, 64, 512)] == [A.form(N, mc.Options(spmm_merge=-mc.SPMM_DENSE)) for N in (16, 64, 512)]


@pytest.mark.parametrize("pin", [dict(spmm_stages=1), dict(spmm_splitting=-1), dict(spmm_slab_waves=8), dict(spmm_slab_panels=2),
                                 dict(spmm_slab=-1), dict(spmm_row_tile_bytes=128), dict(spmm_waves=4)])
def test_options_of_the_other_forms_rule_out_the_copy_with_all_columns(A, pin):
    """What pins part of another form is run in one of them, unless the copy with all columns is asked for beside what it can ignore."""
    L, o = host.load(), mc.Options(**pin)
    kernel, detail = A.run(512, o, ex=True)
    assert kernel != "dense" and A.form(512, o) < 4
    assert kernel != "gather" or detail == pin.get("spmm_stages", 2)
    L.mc_set_thread_options(o)
    assert A.run(512)[0] == kernel
    asked = A.run(512, mc.Options(spmm_merge=mc.SPMM_DENSE, **pin), ex=True)[0]
    assert (asked == "dense") == (not pin.keys() & {"spmm_slab", "spmm_row_tile_bytes", "spmm_waves"})


def test_options_that_say_what_is_automatic_are_no_pins(A):
    """Two chunks in flight and the sharing of long panels are the defaults that the one-knob setters go back to."""
    L = host.load()
    assert L.mc_set_spmm_stages(1) == 0 and L.mc_set_spmm_splitting(0) == 0
    assert A.run(512)[0] != "dense"
    assert L.mc_set_spmm_stages(2) == 0 and L.mc_set_spmm_splitting(1) == 0
    assert A.run(512)[0] == "dense" and A.form(512, mc.Options(spmm_stages=2, spmm_splitting=1)) == 6


@pytest.mark.parametrize("shape", [DENSE, dict(M=4096, K=4096, V=2, empty=0.5), dict(M=1024, K=2048, V=4, empty=0.5, prec="L8R4"),
                                   dict(M=1024, K=1024, V=2, empty=0.5, prec="L16R8")])
def test_the_copy_with_all_columns_replaces_no_other_copy(shape):
    """Calls that ask for another form get the one that they get from an operand built without that copy."""
    A, without = host.Mat(**shape), host.Mat(**shape, options=mc.Options(spmm_merge=-mc.SPMM_DENSE))
    assert any(A.form(N) & 4 for N in (128, 256, 512, 1024)) and not any(without.form(N) & 4 for N in (128, 256, 512, 1024))
    for N in (64, 128, 256, 512, 1024):
        for o in (dict(spmm_slab=1), dict(spmm_slab=-1), dict(spmm_merge=1), dict(spmm_merge=-1), dict(spmm_merge=1, spmm_slab=1), dict(spmm_stages=1),
                  dict(spmm_merge=-mc.SPMM_DENSE)):
            o = mc.Options(**o)
            assert A.form(N, o) == without.form(N, o) and A.run(N, o, ex=True) == without.run(N, o, ex=True)
    A.close(), without.close()


@pytest.mark.parametrize("asked", [False, True])
@pytest.mark.parametrize("used", [False, True])
def test_new_values_refill_the_copy_with_all_columns_only_where_it_is_read(asked, used):
    """An operand whose copy was neither asked for nor read gets its new values in the other formats, and products take their forms
    from then on.  A product that read it may sit in a graph, which will read it again: it is kept up to date."""
    L = host.load()
    A = host.Mat(**DENSE, options=mc.Options(spmm_merge=mc.SPMM_DENSE) if asked else None)
    without = host.Mat(**DENSE, options=mc.Options(spmm_merge=-mc.SPMM_DENSE))
    other = mc.Options(spmm_merge=-mc.SPMM_DENSE)
    assert A.form(512) == 6 and A.run(512, other, ex=True)[0] != "dense" # (neither reads the copy)
    if used:
        assert A.run(512)[0] == "dense"
    for _ in range(2):
        assert L.mc_mat_set_values_device(A.handle, A.values.ctypes.data, None) == 0
        assert L.host_called() == (b"fill" if asked or used else b"values")
        for N in (32, 64, 128, 512, 1024):
            assert (A.form(N) >= 4) == (A.run(N)[0] == "dense")
            assert asked or used or (A.run(N) == without.run(N) and A.form(N) == without.form(N))
        assert (asked or used) == (A.run(512)[0] == "dense") == (A.run(512, mc.Options(spmm_merge=mc.SPMM_DENSE), ex=True)[0] == "dense")
    A.close(), without.close()


def test_an_operand_without_memory_for_the_copy_with_all_columns():
    """The copy is optional: an operand that is built where it does not fit runs in the other forms, and holds nothing of it."""
    L = host.load()
    asked = mc.Options(spmm_merge=mc.SPMM_DENSE)
    shape = dict(M=512, K=4096, V=8, empty=0.9, options=asked)
    with_it = host.Mat(**shape)
    assert with_it.form(512, asked) & 4
    full = L.host_live()
    with_it.close()
    L.host_limit(512 * 4096)                                          # (the copy's size; all else is smaller)
    try:
        A = host.Mat(**shape)
        assert L.host_live() == full - 1
        assert A.form(512, asked) < 4 and A.run(512, asked, ex=True)[0] != "dense"
        assert L.mc_mat_set_values_device(A.handle, A.values.ctypes.data, None) == 0 and L.host_called() == b"values"
        assert A.form(512, asked) < 4
        A.close()
        L.host_limit(1024)                                            # what the operand needs is still asked for
        host.Mat(**shape, status=mc.MC_EHIP)
    finally:
        L.host_limit(2**62)
    assert L.host_live() == 0
