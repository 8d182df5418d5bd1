"""The library's host code (argument checks, options, copies of an operand, choice of form) as a library of its own that runs
without a GPU: api.hip and format_host.cpp by the host compiler, device memory from malloc, and launchers that only write down
which of them was called last.  hipMalloc of `limit` bytes and more fails; live() counts the allocations."""
import ctypes
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from paper_2209_06979_amd import binding as mc

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_06979_amd", "csrc")
STUBS = r"""
#include "attention_order.h"
#include "internal.h"
#include <atomic>
#include <cstdlib>
#include <cstring>
static std::atomic<size_t> limit{~(size_t)0};
static std::atomic<long> allocations{0};
static thread_local char called[64] = "";
static thread_local int detail = 0, variant[2] = {0, 0};
static thread_local int heads_waves[8][3], n_attention = 0;
static hipError_t note(const char *what, int d = 0) { strcpy(called, what); detail = d; return hipSuccess; }
static hipError_t attention(const AttnArgs &a, int heads, int waves, int head_bytes)
{
    if (n_attention < 8) {
        heads_waves[n_attention][0] = heads; heads_waves[n_attention][1] = waves;
        heads_waves[n_attention][2] = attention_pair_shift(a, heads, head_bytes);
    }
    ++n_attention;
    return note("attention", 10 * heads + waves);
}
extern "C" {
void host_limit(size_t bytes) { limit = bytes; }
long host_live() { return allocations; }
const char *host_called() { return called; }
int host_detail() { return detail; }
int host_variant(int i) { return variant[i]; }
int host_attention(int i, int what) { return heads_waves[i][what]; }
int host_attentions() { const int n = n_attention; n_attention = 0; return n; }
hipError_t hipMalloc(void **p, size_t n)
{
    if (n >= limit) return *p = nullptr, hipErrorOutOfMemory;
    ++allocations;
    return *p = malloc(n ? n : 1), hipSuccess;
}
hipError_t hipFree(void *p) { if (p) --allocations; free(p); return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { return memcpy(d, s, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}
hipError_t launch_spmm(mc_prec, const SpmmArgs &a, int bnb, int waves, hipStream_t)
{
    variant[0] = bnb; variant[1] = waves;
    return note("gather", a.stages);
}
hipError_t launch_spmm_slab(mc_prec, const SlabArgs &, int nt, hipStream_t) { return note("lds", nt); }
hipError_t launch_spmm_dense(mc_prec, const DenseArgs &, int tile, hipStream_t) { return note("dense", tile); }
hipError_t launch_dense_fill(const DenseFillArgs &, hipStream_t) { return note("fill"); }
hipError_t launch_set_values(ValuesArgs a, hipStream_t) { return note("values", a.njobs); }
hipError_t launch_zero_rows(int32_t *, int64_t, int, int, const int32_t *, int, hipStream_t) { return note("zero rows"); }
hipError_t launch_zero_ints(int32_t *, int64_t, hipStream_t) { return note("zero"); }
hipError_t launch_spmm_phase_probe(const SpmmArgs &, hipStream_t) { return note("probe"); }
hipError_t launch_gather_probe(const SpmmArgs &, int, int, int32_t *, hipStream_t) { return note("probe"); }
hipError_t launch_mfma_probe(int, int, int32_t *, hipStream_t) { return note("probe"); }
hipError_t launch_finish_split_rows(const int32_t *, int, int, int, int, const int32_t *, void *, int64_t, int64_t, int, float, hipStream_t) { return note("finish"); }
hipError_t launch_sddmm(int, const SddmmArgs &, int, hipStream_t) { return note("sddmm"); }
hipError_t launch_softmax(const SoftmaxArgs &, hipStream_t) { return note("softmax"); }
hipError_t launch_scores_softmax(const ScoresArgs &, int, int, int, hipStream_t) { return note("scores"); }
int scores_softmax_max_npad(int, int) { return 4096; }
hipError_t launch_absmax(const float *, int64_t, float *, hipStream_t) { return note("absmax"); }
hipError_t launch_quantize(const float *, int64_t, float, int, uint8_t *, hipStream_t) { return note("quantize"); }
hipError_t launch_attention_fused(const AttnArgs &a, int heads, int waves, int, int bits, int dk, hipStream_t) { return attention(a, heads, waves, dk * bits / 8); }
hipError_t launch_attention_fused_padded(const AttnArgs &a, int heads, int waves, int, int, int, hipStream_t) { return attention(a, heads, waves, a.real_pieces * 16); }
int attention_fused_max_vectors() { return 4096; }
"""
_lib = None


def load():
    """The library (built once per process), or a skip where it cannot be built."""
    global _lib
    if _lib is None:
        cxx = shutil.which("g++")
        if not cxx or not os.path.isdir("/opt/rocm/include/hip"):
            pytest.skip("no host compiler, or no HIP headers")
        with tempfile.TemporaryDirectory() as d:
            with open(os.path.join(d, "stubs.cpp"), "w") as f:
                f.write(STUBS)
            out = os.path.join(d, "libhost.so")
            subprocess.run([cxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=static_cast<const void *>(x)",
                            "-I/opt/rocm/include", f"-I{CSRC}", "-x", "c++", os.path.join(CSRC, "api.hip"), os.path.join(CSRC, "format_host.cpp"),
                            os.path.join(d, "stubs.cpp"), "-o", out], check=True)
            _lib = ctypes.CDLL(out)
        _lib.host_called.restype = ctypes.c_char_p
        _lib.host_live.restype = ctypes.c_long
        _lib.host_limit.argtypes = [ctypes.c_size_t]
        _lib.mc_mat_create.argtypes, _lib.mc_mat_destroy.argtypes = mc.lib.mc_mat_create.argtypes, [ctypes.c_void_p]
        _lib.mc_mat_destroy.restype = None
        for name in ("mc_spmm", "mc_spmm_ex", "mc_spmm_form", "mc_spmm_form_us", "mc_mat_set_values_device", "mc_sparse_attention_ex"):
            getattr(_lib, name).argtypes = getattr(mc.lib, name).argtypes
        _lib.mc_spmm_form_us.restype = ctypes.c_double
        _lib.mc_set_thread_options.argtypes = _lib.mc_get_thread_options.argtypes = [ctypes.POINTER(mc.Options)]
    return _lib


class Mat:
    """An operand of random columns in that library (freed by close).  sigma: of the logarithm of the panels' lengths."""

    def __init__(self, M, K, V, empty, prec="L8R8", options=None, status=0, sigma=0.0):
        L = load()
        rng = np.random.default_rng(M + K)
        keep = np.full(M // V, max(1, round((1 - empty) * K)))
        if sigma:
            lengths = rng.lognormal(0.0, sigma, M // V)
            keep = np.clip(np.rint(lengths / lengths.mean() * keep), 1, K).astype(np.int64)
        self.row_ptr = np.concatenate([[0], np.cumsum(keep)]).astype(np.int32)
        col_idx = np.concatenate([np.sort(rng.permutation(K)[:n]) for n in keep]).astype(np.int32)
        bits = mc.LHS_BITS[prec]
        self.values = np.ones((len(col_idx), V * (16 if bits == 12 else bits) // 8), np.uint8)
        self.K, self.M, self.prec, self.handle = K, M, mc.PREC[prec], ctypes.c_void_p()
        self.rhs = mc.RHS_BITS[prec]
        assert L.mc_set_thread_options(options) == 0
        try:
            rc = L.mc_mat_create(M, K, V, bits, mc._p32(self.row_ptr), mc._p32(col_idx), self.values.ctypes.data, None, ctypes.byref(self.handle))
        finally:
            L.mc_set_thread_options(None)
        assert rc == status

    def form(self, N, options=None):
        """4: with all columns, else 1 (in LDS) and 2 (merged) added up."""
        return load().mc_spmm_form(self.handle, N, self.prec, options)

    def us(self, N, options=None):
        """The time expected of the form that a call takes."""
        return load().mc_spmm_form_us(self.handle, N, self.prec, 4, options)

    def run(self, N, options=None, ex=False, flags=0, ld=None):
        """The kernel that a call launches, and its detail: chunks in flight, segments or tile."""
        L, ld = load(), ld or N
        one = np.zeros(64, np.uint8)                                   # (never read: an aligned address)
        at = one.ctypes.data + -one.ctypes.data % 16
        rc = (L.mc_spmm_ex(self.handle, at, N, ld, self.prec, flags, options, at, N, None) if ex else
              L.mc_spmm(self.handle, at, N, ld, self.prec, at, N, None))
        assert rc == 0
        return L.host_called().decode(), L.host_detail()

    def variant(self, N, options=None, **kw):
        """The tile and the waves of the gathered kernel that a call launches."""
        assert self.run(N, options, ex=True, **kw)[0] == "gather"
        return load().host_variant(0), load().host_variant(1)

    def close(self):
        load().mc_mat_destroy(self.handle)


class Mask:
    """A mask of panels of 8 rows with `lengths` stored vectors each in that library."""

    def __init__(self, L, lengths):
        lib = load()
        self.L, self.handle = L, ctypes.c_void_p()
        row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
        col_idx = np.concatenate([np.arange(n) for n in lengths]).astype(np.int32)
        assert lib.mc_mat_create(L, L, 8, 0, mc._p32(row_ptr), mc._p32(col_idx), None, None, ctypes.byref(self.handle)) == 0

    def attention(self, batch, heads, dk, p_bits=8, qkv_bits=8, token_major=True, options=None, s_p=0.1):
        """(heads, waves) of every fused launch of a layer on this mask."""
        return [(h, w) for h, w, _ in self.launches(batch, heads, dk, p_bits, qkv_bits, token_major, options, s_p)]

    def launches(self, batch, heads, dk, p_bits=8, qkv_bits=8, token_major=True, options=None, s_p=0.1, places=(0, 0), wider=0):
        """The same with log2 of the pairs worked on at a time.  places: of K and V, 16-byte pieces from the start of a line; wider: elements that tokens are longer by."""
        lib, one = load(), np.zeros(512, np.uint8)
        at = one.ctypes.data + -one.ctypes.data % 128
        lib.host_attentions()
        token = heads * dk + wider
        strides = (token * self.L, dk, token) if token_major else (heads * self.L * dk, self.L * dk, dk)
        assert lib.mc_sparse_attention_ex(at, at + 16 * places[0], at + 16 * places[1], batch, heads, self.L, dk, *strides, self.handle, p_bits, qkv_bits, 0.1, 0.1, 0.1, s_p,
                                          0, options, at, None, 0, None) == 0
        return [tuple(lib.host_attention(i, what) for what in range(3)) for i in range(lib.host_attentions())]

    def close(self):
        load().mc_mat_destroy(self.handle)
