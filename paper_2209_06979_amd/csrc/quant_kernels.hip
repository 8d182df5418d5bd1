// First step of the quantized attention layer (paper, Section 5.3): symmetric per-tensor
// quantisation of the projections' fp32 output to int8 or packed int4 codes.
//   absmax:   max |x| over the tensor (the scale is max|x| / qmax, taken by the caller)
//   quantize: q = clamp(rint(x / scale), -qmax, qmax), ties to even.
// Both are single passes over the tensor, 16 bytes per lane and load: pure HBM streaming.
// The code decision is taken as in double precision: an fp32 quotient decides unless it lies
// within 1e-3 of a rounding boundary, and only those lanes repeat the division in fp64.
#include "internal.h"

#include <atomic>
#include <type_traits>

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

__global__ void absmax_init_kernel(float *result) { *result = 0.f; }

// Where the workgroups of a launch leave their maxima for the first one to gather: a row of words that hold the launch's number
// above the 31 bits of a non-negative float.  A word only grows, and value and number arrive together, so that nothing else
// has to be ordered: a word with this launch's number is this launch's maximum, a smaller one is still to come, and a larger one says
// that a later launch has been given the same row (rows go round; launches of many streams can overtake each other).  The first
// workgroup then reduces the whole tensor by itself, and so it does if the others have not run for a long while: it
// never waits for good.  Nothing is tied to a stream, nothing has to be given back.
constexpr int ABSMAX_ROWS = 64, ABSMAX_GROUPS = 256, ABSMAX_POLLS = 1 << 16;
__device__ unsigned long long absmax_words[ABSMAX_ROWS][ABSMAX_GROUPS];

// Workgroups of 1024 threads with four independent 16-byte loads in flight per lane, 64 KB a workgroup and turn; each
// streams one contiguous span.  The loads are non-temporal.
// ALONE: one workgroup has the whole tensor and writes the result.  Otherwise with a number the first workgroup
// gathers what the others left in the number's row; without one (0) they meet in the result itself, which a kernel before this
// one has set to zero.
// Calls back to back: 1 MB 9.4 us as two launches, 4.1 in one; 8 MB 15.2 and 4.2; 24 MB 4.9, 64 MB 26 and 10.4; 512 MB 80 and 78 (6.9 TB/s).  With counters
// of the workgroups that had left their maximum, ordered by waits, one launch took 4.3, 4.9, 6.1, 11.7 and 78.5 us, and with agent-scope
// fences around the counting 5.4, 7.6, 9.6, 15.2 and 82.6.
template <bool ALONE> __global__ __launch_bounds__(1024) void absmax_kernel(const float *x, int64_t n, float *result, unsigned long long number)
{
    constexpr int U = 4;
    const v4f *xv = reinterpret_cast<const v4f *>(x);
    const int64_t nv = n / 4, per = ((nv + gridDim.x - 1) / gridDim.x + 63) & ~(int64_t)63; // (whole kilobytes)
    __shared__ float red[16];
    __shared__ bool gathered;
    float m = 0.f;
    auto take = [&](v4f v) { m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)))); };
    auto stream = [&](int64_t b, int64_t e) {
        int64_t i = b + threadIdx.x;
        for (; i + (U - 1) * 1024 < e; i += U * 1024) {
            v4f v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(&xv[i + u * 1024]);
#pragma unroll
            for (int u = 0; u < U; ++u) take(v[u]);
        }
        if (i < e) { // (the rest at once, too: what is beyond the end repeats the first element of this lane)
            v4f v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(&xv[i + u * 1024 < e ? i + u * 1024 : i]);
#pragma unroll
            for (int u = 0; u < U; ++u) take(v[u]);
        }
    };
    auto reduce = [&]() { // the workgroup's maximum, in its first wave
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 16; ++w) m = fmaxf(m, red[w]);
    };
    const int64_t b = (int64_t)blockIdx.x * per;
    stream(b, (b + per < nv) ? b + per : nv);
    if (blockIdx.x == 0 && threadIdx.x < (unsigned)(n - nv * 4)) m = fmaxf(m, fabsf(x[nv * 4 + threadIdx.x]));
    reduce();
    if (ALONE) {
        if (threadIdx.x == 0) *result = m;
        return;
    }
    // (non-negative floats order like their bit patterns)
    if (number == 0) {
        unsigned *to = reinterpret_cast<unsigned *>(result);
        if (threadIdx.x == 0 && __float_as_uint(m) > __atomic_load_n(to, __ATOMIC_RELAXED)) atomicMax(to, __float_as_uint(m));
        return;
    }
    unsigned long long *row = absmax_words[number % ABSMAX_ROWS];
    if (blockIdx.x != 0) {
        if (threadIdx.x == 0) (void)__hip_atomic_fetch_max(&row[blockIdx.x], number << 31 | __float_as_uint(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (threadIdx.x < 64) {
        bool all = false, mine = true;
        for (int poll = 0; poll < ABSMAX_POLLS && !all; ++poll) {
            bool there = true;
            unsigned long long w[ABSMAX_GROUPS / 64];
#pragma unroll
            for (int q = 0; q < ABSMAX_GROUPS / 64; ++q) {
                const unsigned g = threadIdx.x + 64 * q;
                w[q] = (g == 0 || g >= gridDim.x) ? number << 31 : __hip_atomic_load(&row[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int q = 0; q < ABSMAX_GROUPS / 64; ++q) {
                there = there && (w[q] >> 31) >= number;
                mine = mine && (w[q] >> 31) <= number;
                if ((w[q] >> 31) == number) m = fmaxf(m, __uint_as_float((unsigned)w[q] & 0x7fffffffu));
            }
            all = __all(there);
        }
        const bool ok = __all(all && mine);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if (threadIdx.x == 0) {
            gathered = ok;
            if (ok) *result = m;
        }
    }
    __syncthreads();
    if (gathered) return;
    stream(0, nv);
    reduce();
    if (threadIdx.x == 0) *result = m;
}

// inv = 1 / scale rounded to fp32.  x * inv is within 1.5 units in the last place of x / scale,
// i.e. within 2e-5 for every quotient that is not clamped anyway, far inside the 1e-3 window in
// which the decision is handed to fp64.
__device__ __forceinline__ bool near_tie(float r) { return fabsf(fabsf(r - truncf(r)) - 0.5f) < 1e-3f; }
__device__ __forceinline__ int clamped(float q, float qmax) { return (int)fminf(fmaxf(q, -qmax), qmax); }
__device__ __forceinline__ int code_of(float x, float scale, float inv, float qmax)
{
    const float r = x * inv;
    return clamped(near_tie(r) ? (float)rint((double)x / (double)scale) : rintf(r), qmax); // near a tie: decide in fp64
}

// L loads of 4 elements per lane and unit, one store of their codes.  Each workgroup owns a contiguous span and keeps four units in
// flight per lane (two of what remains); one test for a tie covers four elements.  The codes are what the caller's next kernel reads: they are
// stored past the caches (STREAM, and then two loads a unit: wider stores) only where they would not stay there (QUANTIZE_CACHED).
// The tensor is read past the caches unless it is small (KEEP: below QUANTIZE_KEPT), when it does not drive the codes out and a
// tensor that is quantised again is still there.  int8, three tensors and the attention layer that reads them, replayed from a graph, tensors written
// just before / once and for all, against stores and (up to 128 MB) loads of the respective other kind, two loads a unit and a test for each element:
//   3 x  4 MB  26.9 -> 25.7 / 18.4 -> 17.5 us (token-major; tensors read past the caches 26.1 / 19.8)
//   3 x  8 MB  40.1 -> 38.5 / 28.2 -> 27.0
//   3 x 16 MB  61.6 -> 54.4 / 38.6 -> 37.0 (tensors read through the caches 59.2 / 36.1)
// By itself, eight tensors in turn: 1 MB 2.4 both, 4 MB 3.0 -> 3.1, 16 MB 5.4 -> 6.1, 32 MB 8.7 -> 9.2, 64 MB 17.3 -> 15.7, 128 MB 30.7 -> 29.5,
// 256 MB 59.8 -> 58.2, 512 MB 111 both (5.9 TB/s).
template <int BITS, bool STREAM, bool KEEP> __global__ __launch_bounds__(256) void quantize_kernel(const float *x, int64_t n, float scale, uint8_t *q)
{
    constexpr int U = 4, L = STREAM ? 2 : 1;
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    typedef typename std::conditional<BITS * L == 16, v2u, typename std::conditional<BITS * L == 8, unsigned, unsigned short>::type>::type Word;
    const float qmax = (BITS == 8) ? 127.f : 7.f, inv = 1.f / scale;
    const v4f *xv = reinterpret_cast<const v4f *>(x);
    const int64_t nu = n / (4 * L), per = ((nu + gridDim.x - 1) / gridDim.x + 63) & ~(int64_t)63; // (whole kilobytes)
    const int64_t b = (int64_t)blockIdx.x * per, e = (b + per < nu) ? b + per : nu;
    auto codes = [&](v4f v) -> unsigned {
        const v4f r = {v.x * inv, v.y * inv, v.z * inv, v.w * inv};
        v4f c = {rintf(r.x), rintf(r.y), rintf(r.z), rintf(r.w)};
        if (near_tie(r.x) || near_tie(r.y) || near_tie(r.z) || near_tie(r.w)) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (near_tie(r[t])) c[t] = (float)rint((double)v[t] / (double)scale);
        }
        unsigned w = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) w |= (unsigned)(clamped(c[t], qmax) & (BITS == 8 ? 255 : 15)) << (BITS * t); // int4: element 2j in bits 3:0 of byte j
        return w;
    };
    auto emit = [&](int64_t i, const v4f (&v)[L]) {
        Word w;
        if constexpr (L == 1) w = (Word)codes(v[0]);
        else if constexpr (BITS == 8) w = (Word){codes(v[0]), codes(v[L - 1])};
        else w = codes(v[0]) | codes(v[L - 1]) << 16;
        Word *to = reinterpret_cast<Word *>(q) + i;
        if (STREAM) __builtin_nontemporal_store(w, to);
        else *to = w;
    };
    auto load = [&](int64_t i, v4f (&v)[L]) {
#pragma unroll
        for (int l = 0; l < L; ++l) v[l] = KEEP ? xv[i * L + l] : __builtin_nontemporal_load(&xv[i * L + l]);
    };
    int64_t i = b + threadIdx.x;
    for (; i + (U - 1) * 256 < e; i += U * 256) {
        v4f v[U][L];
#pragma unroll
        for (int u = 0; u < U; ++u) load(i + u * 256, v[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) emit(i + u * 256, v[u]);
    }
    if (i + 256 < e) { // (two of two or three more)
        v4f v[2][L];
        load(i, v[0]);
        load(i + 256, v[1]);
        emit(i, v[0]);
        emit(i + 256, v[1]);
        i += 512;
    }
    if (i < e) {
        v4f v[L];
        load(i, v);
        emit(i, v);
    }
    // tail of fewer than 4 L elements (n is even for 4-bit codes)
    if (blockIdx.x == 0) {
        const int64_t t0 = nu * 4 * L;
        if (BITS == 8) {
            if (threadIdx.x < (unsigned)(n - t0)) q[t0 + threadIdx.x] = (uint8_t)(code_of(x[t0 + threadIdx.x], scale, inv, qmax) & 255);
        } else if (threadIdx.x < (unsigned)((n - t0) / 2)) {
            const int64_t e = t0 + 2 * threadIdx.x;
            q[e / 2] = (uint8_t)((code_of(x[e], scale, inv, qmax) & 15) | ((code_of(x[e + 1], scale, inv, qmax) & 15) << 4));
        }
    }
}

constexpr int64_t QUANTIZE_CACHED = 32 << 20; // bytes of codes: an eighth of the memory-side cache
constexpr int64_t QUANTIZE_KEPT = 8 << 20;    // bytes of the tensor

// units of 256 threads' worth of work, at most `cap` workgroups
inline unsigned grid_for(int64_t units, int64_t cap)
{
    const int64_t blocks = (units + 255) / 256;
    return (unsigned)(blocks < 1 ? 1 : (blocks > cap ? cap : blocks));
}

} // namespace

// The number of a launch on the stream's device (they count from 1).  0: the launch may run several times under its number (while a
// graph is captured), the device is not known, or the numbers' 33 bits are used up.
static unsigned long long absmax_number(hipStream_t s)
{
    constexpr int DEVICES = 64;
    static std::atomic<unsigned long long> launches[DEVICES];
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    int dev = -1;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone ||
        (s ? hipStreamGetDevice(s, &dev) : hipGetDevice(&dev)) != hipSuccess || dev < 0 || dev >= DEVICES) {
        (void)hipGetLastError();
        return 0;
    }
    const unsigned long long number = launches[dev].fetch_add(1, std::memory_order_relaxed) + 1;
    return number >> 33 ? 0 : number;
}

hipError_t launch_absmax(const float *x, int64_t n, float *result, hipStream_t s)
{
    // a workgroup takes 64 KB at a time; one on every compute unit saturates the memory (more only take longer to meet), and
    // one alone reads 128 KB sooner than two have met
    const int64_t groups = (n + 16383) / 16384;
    if (groups <= 2) { // (also an empty tensor)
        return launch_kernel((absmax_kernel<true>), dim3(1), dim3(1024), 0, s, x, n, result, 0ull);
    }
    const unsigned long long number = absmax_number(s);
    if (number == 0) {
        const hipError_t e = launch_kernel(absmax_init_kernel, dim3(1), dim3(1), 0, s, result);
        if (e != hipSuccess) return e;
    }
    return launch_kernel((absmax_kernel<false>), dim3((unsigned)(groups < ABSMAX_GROUPS ? groups : ABSMAX_GROUPS)), dim3(1024), 0, s, x, n, result, number);
}

hipError_t launch_quantize(const float *x, int64_t n, float scale, int bits, uint8_t *q, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    // a load per lane as long as that makes no more than 2048 workgroups, then up to eight
    const int64_t loads = n / 4 / 256;
    const dim3 grid(grid_for(n / 4, loads <= 2048 ? 2048 : loads / 8 < 2048 ? 2048 : loads / 8 < 16384 ? loads / 8 : 16384)), block(256);
    const bool stream = n * bits / 8 > QUANTIZE_CACHED, keep = n * 4 < QUANTIZE_KEPT;
    if (bits == 8 && stream) return launch_kernel((quantize_kernel<8, true, false>), grid, block, 0, s, x, n, scale, q);
    if (bits == 8 && keep) return launch_kernel((quantize_kernel<8, false, true>), grid, block, 0, s, x, n, scale, q);
    if (bits == 8) return launch_kernel((quantize_kernel<8, false, false>), grid, block, 0, s, x, n, scale, q);
    if (stream) return launch_kernel((quantize_kernel<4, true, false>), grid, block, 0, s, x, n, scale, q);
    if (keep) return launch_kernel((quantize_kernel<4, false, true>), grid, block, 0, s, x, n, scale, q);
    return launch_kernel((quantize_kernel<4, false, false>), grid, block, 0, s, x, n, scale, q);
}
