// New values for an operand, from interchange order into every device format it has, in one launch: its panels, its
// LDS-ordered copy, and the same two of its merged copy.  (It was a launch per format and one for the merged values in
// interchange order: with the first kernels of a layer's steps that is what a small layer waits for.)
//
// What bounds it: latency -- the formats of 100,000 vectors are a few megabytes -- so a wave takes one chunk of one format, and
// its chain is short: the chunk's first vector (one scalar load), for a merged panel the vectors behind its shares, their values, one
// trip through LDS.  A lane has one slot: the bytes of up to eight of its rows are one 64-bit LDS write, the transposing read gives
// a lane eight slots of one row, and those 8 bytes are the format's.  Waves never meet.
// 2048 x 2048, 90 % empty, V = 8 (panels, merged panels and their LDS-ordered copy), under the profiler: a launch per format 18 us;
// one launch, the panel looked up, bytes put into place one by one and workgroups that meet 5.1; as it is 4.1.
#include "internal.h"
#include "lds_async.h"

namespace {

using mcu::v2i;
// (a caller's values have no particular alignment)
struct __attribute__((packed, aligned(1))) u16_any { uint16_t x; };
struct __attribute__((packed, aligned(1))) u32_any { uint32_t x; };
struct __attribute__((packed, aligned(1))) u64_any { uint64_t x; };

// byte 0 .. 3 of x and of y in turn: the first two of each, the last two
__device__ __forceinline__ uint64_t interleaved(uint32_t x, uint32_t y)
{
    return (uint64_t)__builtin_amdgcn_perm(y, x, 0x07030602) << 32 | __builtin_amdgcn_perm(y, x, 0x05010400);
}

// V values of `bits` each from s
template <int BYTES> __device__ __forceinline__ void load_vector(const uint8_t *s, uint64_t &x, uint64_t &y)
{
    y = 0;
    if constexpr (BYTES == 1) x = *s;
    else if constexpr (BYTES == 2) x = reinterpret_cast<const u16_any *>(s)->x;
    else if constexpr (BYTES == 4) x = reinterpret_cast<const u32_any *>(s)->x;
    else x = reinterpret_cast<const u64_any *>(s)->x;
    if constexpr (BYTES == 16) y = reinterpret_cast<const u64_any *>(s + 8)->x;
}

// V: rows of a stored vector
template <int BITS, int V> __global__ __launch_bounds__(256) void set_values_kernel(ValuesArgs a)
{
    constexpr int PL = BITS == 16 ? 2 : 1;                       // byte planes
    constexpr int VB = V * BITS / 8, MOST = 8 / V;               // bytes of a vector; vectors that eight rows come from, at most
    __shared__ __attribute__((aligned(16))) uint64_t stage[4][PL][MC_CHUNK];
    int k = 0;
    while (k + 1 < a.njobs && (int)blockIdx.x >= a.job[k + 1].first_block) ++k;
    const ValuesJob &job = a.job[k];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, l = lane & 15;
    const int64_t chunk = (int64_t)(blockIdx.x - job.first_block) * 4 + w;
    if (chunk >= job.nchunks) return;
    int64_t vec = -1;                                            // the stored vector of this lane's slot, -1: padding
    if (job.blk_src) {
        vec = job.blk_src[chunk * MC_CHUNK + lane];
    } else {
        const v2i c = *reinterpret_cast<const v2i *>(job.chunk_vec + 2 * chunk);
        if (lane < c.y) vec = c.x + lane;
    }
    const int rows = job.V, shares = rows / V;                   // a merged vector's rows come from `shares` vectors
    const int octets = rows > 8 ? 2 : 1, per = shares / octets;  // rows are handled eight at a time
    // (two chunks in a record: a group of 16 slots of each in turn)
    constexpr int GROUP = BITS == 4 ? 8 : 16 * PL;               // bytes of a row's 16 slots
    const int per_rec = job.rec_chunks;
    uint8_t *const dst = job.dst + (per_rec == 2 ? chunk >> 1 : chunk) * job.rec_bytes + job.head_bytes +
                         (g * per_rec + (per_rec == 2 ? (int)chunk & 1 : 0)) * (GROUP * rows);
    for (int o = 0; o < octets; ++o) {
        // all sources, then all values: each a round trip to memory
        int64_t from[MOST];
#pragma unroll
        for (int q = 0; q < MOST; ++q) from[q] = q == 0 ? vec : -1;
        if (job.merge_src) {
#pragma unroll
            for (int q = 0; q < MOST; ++q) from[q] = (q < per && vec >= 0) ? job.merge_src[vec * shares + o * per + q] : -1;
        }
        uint64_t x[MOST], y[MOST], bytes[PL] = {};               // row r of the eight in byte r
#pragma unroll
        for (int q = 0; q < MOST; ++q) load_vector<VB>(a.src + (from[q] < 0 ? 0 : from[q]) * VB, x[q], y[q]);
#pragma unroll
        for (int q = 0; q < MOST; ++q) {
            if (from[q] < 0) x[q] = y[q] = 0;
            constexpr uint32_t NIB = 0x0F0F0F0Fu;
            const int at = 8 * V * q;
            if constexpr (BITS == 8) {
                bytes[0] |= x[q] << at;
            } else if constexpr (BITS == 4) {
                bytes[0] |= interleaved((uint32_t)x[q] & NIB, (uint32_t)(x[q] >> 4) & NIB) << at;
            } else { // value = 256 * high + low, both signed: the low byte as it is, the high byte of the value + 128
                const uint32_t w4[4] = {(uint32_t)x[q], (uint32_t)(x[q] >> 32), (uint32_t)y[q], (uint32_t)(y[q] >> 32)};
                uint32_t r4[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) r4[t] = ((w4[t] & 0x7FFF7FFFu) + 0x00800080u) ^ (w4[t] & 0x80008000u);
                bytes[PL - 1] |= ((uint64_t)__builtin_amdgcn_perm(w4[3], w4[2], 0x06040200) << 32 | __builtin_amdgcn_perm(w4[1], w4[0], 0x06040200)) << at;
                bytes[0] |= ((uint64_t)__builtin_amdgcn_perm(r4[3], r4[2], 0x07050301) << 32 | __builtin_amdgcn_perm(r4[1], r4[0], 0x07050301)) << at;
            }
        }
#pragma unroll
        for (int p = 0; p < PL; ++p) stage[w][p][lane] = bytes[p];
        mcu::lgkm_wait();                                        // (LDS executes a wave's instructions in order: for the compiler)
        __builtin_amdgcn_wave_barrier();
        // lane l of a group of 16 slots: row l % 8 of the octet, slots 0 .. 7 (l < 8) or 8 .. 15
        const int row = o * 8 + (l & 7), up = l >> 3;
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            v2i d = mcu::lds_read_tr8(&stage[w][p][g * 16 + (l >> 1) + 8 * (l & 1)]);
            if constexpr (BITS == 4) {                           // byte b: slots b and b + 8
                const v2i odd = {__builtin_amdgcn_update_dpp(0, d.x, 0x128, 0xF, 0xF, false), __builtin_amdgcn_update_dpp(0, d.y, 0x128, 0xF, 0xF, false)};
                d = (v2i){d.x | odd.x << 4, d.y | odd.y << 4};
                if (row < rows && up == 0) *reinterpret_cast<v2i *>(dst + row * 8) = d;
            } else if (row < rows) {
                *reinterpret_cast<v2i *>(dst + (p * rows + row) * 16 + up * 8) = d;
            }
        }
        mcu::lgkm_wait();                                        // the next octet goes to the same place
        __builtin_amdgcn_wave_barrier();
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
    const dim3 grid((unsigned)blocks), block(256);
    switch (a.bits * 16 + a.V) {
    case 4 * 16 + 2: return launch_kernel(set_values_kernel<4, 2>, grid, block, 0, s, a);
    case 4 * 16 + 4: return launch_kernel(set_values_kernel<4, 4>, grid, block, 0, s, a);
    case 4 * 16 + 8: return launch_kernel(set_values_kernel<4, 8>, grid, block, 0, s, a);
    case 8 * 16 + 2: return launch_kernel(set_values_kernel<8, 2>, grid, block, 0, s, a);
    case 8 * 16 + 4: return launch_kernel(set_values_kernel<8, 4>, grid, block, 0, s, a);
    case 8 * 16 + 8: return launch_kernel(set_values_kernel<8, 8>, grid, block, 0, s, a);
    case 16 * 16 + 2: return launch_kernel(set_values_kernel<16, 2>, grid, block, 0, s, a);
    case 16 * 16 + 4: return launch_kernel(set_values_kernel<16, 4>, grid, block, 0, s, a);
    case 16 * 16 + 8: return launch_kernel(set_values_kernel<16, 8>, grid, block, 0, s, a);
    default: return hipErrorInvalidValue;
    }
}
