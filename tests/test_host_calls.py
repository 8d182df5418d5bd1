"""Arguments of the extension module's compute calls as far as they can be checked without a GPU."""
import numpy as np
import pytest
import torch

from paper_2209_06979_amd import binding as mc

cpu = torch.zeros((64, 64), dtype=torch.int8)


@pytest.mark.parametrize("call", [mc.spmm, mc.spmm_dequant, mc.sddmm, mc.sddmm_dequant, mc.sddmm_to_mat, mc.absmax, mc.quantize,
                                  mc.sparse_softmax, mc.sparse_softmax_to_mat, mc.sparse_attention, mc.sparse_attention_static])
def test_missing_surplus_and_unknown_arguments(call):
    with pytest.raises(TypeError):
        call()
    with pytest.raises(TypeError):
        call(*([None] * 20))
    with pytest.raises(TypeError):
        call(cpu, cpu, cpu, cpu, 1.0, 1.0, 1.0, 1.0, nothing=1)


def test_wrong_kinds_of_arguments():
    with pytest.raises(AssertionError):
        mc.spmm(None, cpu, "L8R8")                       # not on the device
    with pytest.raises(AssertionError):
        mc.absmax(cpu)
    with pytest.raises(AssertionError):
        mc.quantize(torch.zeros(16), np.float32(0.5))
    with pytest.raises(KeyError):
        mc.sddmm(cpu, cpu, None, "L9R9")
    with pytest.raises(KeyError):
        mc.sddmm_to_mat(Q=cpu, Kmat=cpu, P=None, prec=8, scale=1.0)
    with pytest.raises(TypeError):
        mc.sddmm(cpu, cpu, "mask", "L8" + "R8")          # (a precision that is equal but not the same object)
    with pytest.raises(TypeError):
        mc.spmm(A=None, B="rows", prec="L8R8")
    with pytest.raises(TypeError):
        mc.spmm(None, cpu, "L8R8", A=None)               # given twice


def test_status_of_the_library_becomes_the_bindings_error():
    m = mc.SparseMatrix.__new__(mc.SparseMatrix)         # a closed matrix: no handle
    with pytest.raises(AssertionError):
        m.set_values(cpu)
    m.close()
