"""The sparse softmax at the panel lengths and numbers of panels where another kernel takes over: codes against the oracle, and the
device panel format against the same codes written as values."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import torch_dev
from test_gpu_softmax import _check, _counts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("many", [False, True])              # at most 512 panels in all score sets, or more
@pytest.mark.parametrize("scores", [512, 1024, 2048, 3072, 4096, 8192, 16384])
@pytest.mark.parametrize("V", [2, 4, 8])
def test_lengths_where_the_kernel_changes(V, scores, many):
    """The longest panel at a limit and one vector beyond it (a panel is padded to 64 vectors)."""
    for beyond in (0, 1):
        n = scores // V + beyond
        L = max(-(-n // V) * V, 64 * V)
        counts = _counts(L // V, [n, 0, 1, n - 1, 63], 0)
        if L // V <= 512:
            counts[5:] = 3
        _check(V, L, counts, 7400 + V, 8, batch=max(1, 513 // (L // V) + 1) if many else 1)


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("scores", [512, 1024, 2048, 3072, 4096, 8192, 16384, 16385])
@pytest.mark.parametrize("V,P", [(2, 64), (4, 600), (8, 64), (8, 600)])
def test_device_format_of_every_kernel(V, P, scores, bits):
    import torch
    from paper_2209_06979_amd import binding as mc
    n = -(-scores // V)
    K = max(-(-n // 16) * 16, 128)
    counts = np.r_[[n, 0, 1, n - 1, 65], 2 + np.arange(P - 5) % 7]
    rp, ci = wl.ragged_pattern(V * P, K, V, counts, 7500)
    rng = np.random.default_rng(7501)
    S = torch.from_numpy(rng.integers(-9000, 9000, len(ci) * V).astype(np.int32)).cuda()
    zeros = np.zeros((len(ci), V), np.int8 if bits == 8 else np.int16)
    prec = "L8R8" if bits == 8 else "L16R8"
    B = torch.from_numpy(wl.uniform_int8((K, 64), 7502)).cuda()
    outs = []
    for direct in (True, False):
        A = mc.SparseMatrix(V * P, K, V, rp, ci, zeros, bits)
        if direct:
            mc.sparse_softmax_to_mat(A, S, 2.5e-4, 127.0 if bits == 8 else 32639.0)
        else:
            codes = torch.empty((1, len(ci) * V), dtype=torch.int8 if bits == 8 else torch.int16, device="cuda")
            mc.sparse_softmax(A, S.reshape(1, -1), 2.5e-4, 127.0 if bits == 8 else 32639.0, out=codes, code_bits=bits)
            A.set_values(codes.reshape(len(ci), V))
        outs.append(mc.spmm(A, B, prec, options=mc.Options(spmm_slab=-1, spmm_merge=-1)).cpu().numpy())
        A.close()
    assert np.array_equal(*outs) and outs[0].any()


@pytest.mark.parametrize("scores,units", [(3080, 1536), (3080, 1537), (4096, 1537), (4096, 20481), (4104, 768), (4104, 769), (8192, 1024), (8192, 1025),
                                          (4104, 4097)])
def test_numbers_of_panels_where_the_kernel_changes(scores, units):
    """Few full panels among short ones: the launch is as large, the oracle's work is not."""
    n = scores // 8
    L = -(-n // 8) * 8
    panels = L // 8
    batch = units // panels if units % 2 == 0 else -(-units // panels) # (up to the limit, or beyond it)
    counts = _counts(panels, [n, 0, 1, n - 1, 63], 0)
    counts[5:] = 3
    _check(8, L, counts, 7600, 8, batch=batch)


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("P,scores", [(1600, 4096), (1600, 3080), (800, 4104), (4104, 8192)])
def test_device_format_of_many_panels(P, scores, bits):
    """The splits that only large launches take, in the panel format: single waves of 16 pieces, four waves of 16."""
    test_device_format_of_every_kernel(8, P, scores, bits)
