// New values for an operand, from interchange order into every device format it has, in one launch: its panels, its
// LDS-ordered copy, and the same two of its merged copy.  (It was a launch per format and one for the merged values in
// interchange order: with the first kernels of a layer's steps that is what a small layer waits for.)
//
// What bounds it: latency -- the formats of 100,000 vectors are a few megabytes -- and, written byte by byte as the formats
// ask for it (the values of a vector lie 16 or 8 bytes apart), the number of stores.  A workgroup therefore takes four chunks of
// one format, a thread reads one slot's vector in one or two loads, the bytes are put into place in LDS, and the finished
// chunks are copied out 16 bytes at a time.
// 2048 x 2048, 90 % empty, V = 8 (panels, merged panels and their LDS-ordered copy): 4 launches, 18 us -> 1 launch, 5.8 us
// under the profiler; the layer's steps with it 28.7 -> 16.3 us.
#include "internal.h"

namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));
// (a caller's values have no particular alignment)
struct __attribute__((packed, aligned(1))) u16_any { uint16_t x; };
struct __attribute__((packed, aligned(1))) u32_any { uint32_t x; };
struct __attribute__((packed, aligned(1))) u64_any { uint64_t x; };

__global__ __launch_bounds__(256) void set_values_kernel(ValuesArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t tile[4 * MC_CHUNK * 16];       // four chunks: 64 slots x 16 rows of a byte, or 8 of two planes
    int k = 0;
    while (k + 1 < a.njobs && (int)blockIdx.x >= a.job[k + 1].first_block) ++k;
    const ValuesJob &job = a.job[k];
    const int64_t chunk0 = (int64_t)(blockIdx.x - job.first_block) * 4;
    const int tid = threadIdx.x, i = tid & 63, g = i >> 4, b = i & 15;
    const int64_t chunk = chunk0 + (tid >> 6);
    const int rows = job.V, cbytes = MC_CHUNK * rows * a.bits / 8;
    // the stored vector of this slot, -1: padding
    int64_t vec = -1;
    if (chunk < job.nchunks) {
        if (job.blk_src) {
            vec = job.blk_src[chunk * MC_CHUNK + i];
        } else {
            const int p = job.chunk_panel[chunk], s0 = job.panel_ptr[2 * p];
            const int64_t at = chunk * MC_CHUNK + i - s0;
            if (at < job.panel_ptr[2 * p + 1] - s0) vec = job.row_ptr[p] + at;
        }
    }
    uint8_t *mine = tile + (tid >> 6) * cbytes;
    const int shares = rows / a.V, vb = a.V * a.bits / 8;         // a merged vector's rows come from that many vectors
    for (int q = 0; q < shares; ++q) {
        const int64_t from = (job.merge_src && vec >= 0) ? job.merge_src[vec * shares + q] : vec;
        uint64_t lo = 0, hi = 0;
        if (from >= 0) {
            const uint8_t *s = a.src + from * vb;
            switch (vb) {
            case 1: lo = *s; break;
            case 2: lo = reinterpret_cast<const u16_any *>(s)->x; break;
            case 4: lo = reinterpret_cast<const u32_any *>(s)->x; break;
            case 8: lo = reinterpret_cast<const u64_any *>(s)->x; break;
            default: lo = reinterpret_cast<const u64_any *>(s)->x; hi = reinterpret_cast<const u64_any *>(s + 8)->x; break;
            }
        }
        const int v0 = q * a.V;
        if (a.bits == 8) {
            for (int v = 0; v < a.V; ++v) mine[g * (16 * rows) + (v0 + v) * 16 + b] = (uint8_t)((v < 8 ? lo : hi) >> (8 * (v & 7)));
        } else if (a.bits == 16) {
            for (int v = 0; v < a.V; ++v) {
                const int x = (int16_t)((v < 4 ? lo : hi) >> (16 * (v & 3))), h = (x + 128) >> 8, l = x - h * 256;
                mine[g * (32 * rows) + (v0 + v) * 16 + b] = (uint8_t)h;
                mine[g * (32 * rows) + 16 * rows + (v0 + v) * 16 + b] = (uint8_t)l;
            }
        } else { // slots b and b + 8 share bytes
            const uint64_t other = __shfl_xor((unsigned long long)lo, 8, 64);
            if (b < 8)
                for (int v = 0; v < a.V; ++v) mine[g * (8 * rows) + (v0 + v) * 8 + b] = (uint8_t)(((lo >> (4 * v)) & 15) | (((other >> (4 * v)) & 15) << 4));
        }
    }
    __syncthreads();
    const int per = cbytes / 16;
    for (int u = tid; u < 4 * per; u += 256) {
        const int64_t c = chunk0 + u / per;
        if (c < job.nchunks) *reinterpret_cast<v4u *>(job.dst + c * job.rec_bytes + job.head_bytes + (u % per) * 16) = reinterpret_cast<const v4u *>(tile)[u];
    }
}

} // namespace

hipError_t launch_set_values(ValuesArgs a, hipStream_t s)
{
    int64_t blocks = 0;
    for (int k = 0; k < a.njobs; ++k) {
        a.job[k].first_block = (int)blocks;
        blocks += (a.job[k].nchunks + 3) / 4;
    }
    if (blocks == 0) return hipSuccess;
    return launch_kernel(set_values_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
}
