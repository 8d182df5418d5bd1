"""New values written into every device format of an operand by one launch, and the largest magnitude found by one launch, at
the sizes where their work is split differently."""
import numpy as np
import pytest

from paper_2209_06979_amd import workloads as wl
from gpu_util import torch_dev, run_spmm_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("prec,V", [("L8R8", 2), ("L8R8", 8), ("L4R4", 2), ("L4R4", 4), ("L4R4", 8), ("L16R8", 4), ("L16R8", 8)])
def test_values_reach_every_format(prec, V, offset):
    """Unequal panels (empty ones too), merged and LDS-ordered copies built; values at an address with no alignment beyond
    an element's."""
    import torch
    from paper_2209_06979_amd import binding as mc
    counts = np.r_[[0, 1, 63, 64, 65, 300, 0, 17], np.arange(40) * 7 % 150]
    M, K, N = V * len(counts), 700, 64
    c = wl.spmm_case(M, K, N, V, 0.5, prec, 9300 + V)
    c["row_ptr"], c["col_idx"] = wl.ragged_pattern(M, K, V, counts, 9301)
    n = len(c["col_idx"])

    def values(seed):
        return (wl.uniform_packed_int4((n, V // 2), seed) if prec == "L4R4" else
                wl.uniform_int16((n, V), seed) if prec == "L16R8" else wl.uniform_int8((n, V), seed))
    new = values(9303)
    elem = 2 if prec == "L16R8" else 1
    raw = torch.zeros(new.nbytes + 2, dtype=torch.uint8, device="cuda")
    raw[offset * elem:offset * elem + new.nbytes] = torch.from_numpy(new.reshape(-1).view(np.uint8)).cuda()
    dev = raw[offset * elem:offset * elem + new.nbytes].view(torch.int16 if prec == "L16R8" else torch.int8).reshape(new.shape)
    want = run_spmm_oracle(dict(c, values=new))
    mc.set_thread_options(mc.Options(spmm_slab=1, spmm_merge=1))
    try:
        A = mc.SparseMatrix(M, K, V, c["row_ptr"], c["col_idx"], values(9302), mc.LHS_BITS[prec])
    finally:
        mc.set_thread_options(None)
    A.set_values(dev)
    for merge in (-1, 1):
        for slab in (-1, 1):
            out = torch.full((M, N), -7777777, dtype=torch.int32, device="cuda")
            mc.spmm(A, torch_dev(c["B"]), prec, out=out, options=mc.Options(spmm_merge=merge, spmm_slab=slab))
            assert np.array_equal(out.cpu().numpy(), want), (merge, slab)
    A.close()


@pytest.mark.parametrize("n", [1, 5, 32768, 32769, 32 * 16384 - 3, 32 * 16384 + 1, 256 * 16384 + 777])
def test_absmax_of_interleaved_streams(n):
    """The largest magnitude at either end, several launches in a row on two streams at once."""
    import torch
    from paper_2209_06979_amd import binding as mc
    xs = [torch.randn(n, device="cuda") for _ in range(2)]
    xs[0][0], xs[1][n - 1] = -77.5, 99.25
    outs = [[torch.full((1,), -1.0, device="cuda") for _ in range(6)] for _ in range(2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                mc.absmax(xs[i] if k % 2 == 0 else xs[i][:max(1, n // 2 // 4 * 4)], out=outs[i][k])
    torch.cuda.synchronize()
    for i in range(2):
        half = xs[i][:max(1, n // 2 // 4 * 4)]
        for k in range(6):
            assert float(outs[i][k]) == float((xs[i] if k % 2 == 0 else half).abs().max()), (i, k)


@pytest.mark.parametrize("n", [3 * 16384, 70 * 16384 + 5])
def test_absmax_that_is_overtaken(n):
    """Many streams at once, and a launch that waits on its stream until the 64 later ones after which rows come round again have
    run: its first workgroup finds their numbers in its row."""
    import torch
    from paper_2209_06979_amd import binding as mc
    x = torch.randn(n, device="cuda")
    tops = torch.rand(140, device="cuda") + 50.0
    xs = [x.clone() for _ in range(4)]
    late, want_late = torch.full((1,), -1.0, device="cuda"), float(x.abs().max())
    out = torch.full((140,), -1.0, device="cuda")
    torch.cuda.synchronize()
    held = torch.cuda.Stream()
    with torch.cuda.stream(held):
        torch.cuda._sleep(20_000_000)                          # some ten milliseconds
        mc.absmax(x, out=late)
    streams = [torch.cuda.Stream() for _ in range(35)]
    for k in range(140):
        s = streams[k % 35]
        with torch.cuda.stream(s):
            y = xs[k % 4] * (tops[k] / want_late)
            mc.absmax(y, out=out[k:k + 1])
            y.record_stream(s)
    torch.cuda.synchronize()
    assert float(late) == want_late
    for k in range(140):
        assert float(out[k]) == float((xs[k % 4] * (tops[k] / want_late)).abs().max()), k
