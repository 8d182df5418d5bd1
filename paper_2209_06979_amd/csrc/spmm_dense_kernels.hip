// SpMM on an operand held with all its columns, for patterns whose merged panels name nearly every row of B.
//
// Sixteen rows of a matrix of short vectors, or of a hardly sparse one, have between them an entry in most columns: half
// empty with V = 2 or 4 the union of 16 / V panels is 94 - 99 % of the columns, and three quarters of them at 85 % and V = 2.
// A gather by column index then fetches what a plain product would fetch, but for 16 rows at a time only, because each
// merged panel has its own order of rows of B.  Here the operand's bytes lie in MFMA operand order with zeros where nothing is stored
// (dense_fill_kernel writes them from the panel format), and a workgroup multiplies 32 - 256 rows of it with a column tile of B that
// all of its waves read from LDS.
//
//   A   straight from memory into registers, one 1 KB fragment (16 rows x 64 columns, one byte plane) per load, requested
//       four steps (small tiles: eight) ahead; every fragment is read by one wave of the workgroup only.
//   B   64 rows x NT segments of 16 columns per chunk, loaded into registers seven (small tiles: eleven) steps ahead, written to
//       LDS three steps ahead in the image [row / 16][segment][row % 16] (positions exchanged so that neither the writes nor
//       the transposing reads meet in a bank; nibbles widened to bytes of 16 times their value, once for all waves), read a step
//       ahead.  One barrier per step; it need not wait for anything: what a step overwrites was consumed by the step
//       before, and what it reads was written two steps before, ahead of reads that its writers have waited for since (a
//       wave's writes of a step are issued before its reads, which the kernel sees to).
// The waves of a workgroup are WR row groups times WK groups that take every WK-th chunk; the WK sums meet in LDS at the
// end.  The MFMA computes the transposed tile (as in spmm_resident_kernels.hip): a lane has four neighbouring columns.
//
// What bounds it: the bytes that a compute unit takes in from L2 (48 per clock reached by plain loads): (rows + columns) x K per tile, 24 KB
// in 600 clocks with 128 x 64, of which the MFMAs alone take 290 and with the LDS reads 460; and on the whole chip the clock,
// which falls from 2.4 to 1.7 GHz under this load.  A deeper ring, sixteen waves, four waves of twice the rows, 64 x 128 tiles
// and loads spread among the MFMAs all measured the same within 3 %.
// Whole calls, L8-R8, against the resident form on merged panels (3 operands in turn):
//   4096 x 4096, half empty, V = 2, N = 512          20.6 -> 15.4 us
//   2710 x 7060, 77 % empty, V = 2, N = 272          32.7 -> 18.3
//   4096 x 4096, half empty, V = 2, N = 256          15.4 -> 11.3
// and of 400 drawn operands of all precisions 38 run in this form, 1.24 times as fast in the mean, two of them 1.07 and 1.17 times as long.
#include "internal.h"
#include "lds_async.h"

namespace {

using mcu::v2i;
using mcu::v4f;
using mcu::v4i;
using mcu::lds_v2i;

constexpr int STAGES = 4;

// PL: byte planes of A (2: 16- and 12-bit values).  R4: B holds nibbles.  NT: segments of 16 columns of the column tile.
// RF: blocks of 16 rows per wave.  WR: row groups, W: waves.  AH: steps that operands are requested ahead (the loop is unrolled by
// as many: set and stage numbers are constants).
template <int PL, bool R4, int NT, int RF, int WR, int W, int AH>
__global__ __launch_bounds__(64 * W, PL == 1 && NT == 4 && RF == 2 ? 4 : 1) void spmm_dense_kernel(DenseArgs a)
{
    mcu::request_arguments(a);
    constexpr int WK = W / WR, NP = WK * NT / W, STAGE = WK * NT * 1024, OWN = RF * NT / WK;
    static_assert(NP >= 1 && NP * W == WK * NT && OWN >= 1 && OWN * WK == RF * NT, "whole pieces per thread, whole tiles per wave");
    static_assert(AH % STAGES == 0, "stage numbers repeat with the unrolled loop");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = w % WR, kg = w / WR, j = lane & 15, g = lane >> 4, ii = j >> 1;
    // Workgroups go to the eight XCDs round-robin: each XCD gets a run of tiles, column tiles first, so that its L2 fetches a row
    // of A's fragments once.
    const int tiles = a.tm * a.tn, per = (tiles + 7) / 8, q = blockIdx.x >> 3, t = (blockIdx.x & 7) * per + q;
    if (q >= per || t >= tiles) return;
    const int tm = t / a.tn, col0 = t % a.tn * 16 * NT;

    // ---- operands -----------------------------------------------------------------------------------------
    // (fragments beyond the last row block or chunk: the last one's; rows of B beyond the last are zero by the descriptor's range)
    const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.A), 0, a.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.B), 0, a.b_bytes, 0x00020000);
    int first[RF];
#pragma unroll
    for (int f = 0; f < RF; ++f) {
        const int rb = (tm * WR + rw) * RF + f;
        first[f] = (rb < a.nrb ? rb : a.nrb - 1) * a.nch * (PL * 1024);
    }
    v4i ra[AH][RF][PL];
    auto load_a = [&](int s, int d, int f) {
        const int c = s * WK + kg, at = first[f] + (c < a.nch ? c : a.nch - 1) * (PL * 1024);
#pragma unroll
        for (int p = 0; p < PL; ++p) ra[d][f][p] = __builtin_amdgcn_raw_buffer_load_b128(ar, lane * 16, at + p * 1024, 0);
    };
    unsigned from[NP], to[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int u = tid + 64 * W * i, seg = u % NT, row = u / NT;
        const int col = col0 + seg * 16 < a.cols ? col0 + seg * 16 : col0; // (beyond the last: never stored)
        from[i] = row * (unsigned)a.ldb_bytes + (R4 ? col / 2 : col);
        to[i] = ((row >> 4) * NT + seg) * 256 + (((row & 15) ^ (seg * (8 / NT)) ^ ((row >> 4 & 1) * 8)) * 16);
    }
    const unsigned step_bytes = WK * MC_CHUNK * (unsigned)a.ldb_bytes;
    v4i rb[AH][NP];
    auto load_b = [&](int d) { // (steps in order)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if constexpr (R4) {
                const v2i x = __builtin_amdgcn_raw_buffer_load_b64(br, from[i], 0, 0);
                rb[d][i] = (v4i){x.x, x.y, 0, 0};
            } else {
                rb[d][i] = __builtin_amdgcn_raw_buffer_load_b128(br, from[i], 0, 0);
            }
            from[i] += step_bytes;
        }
    };
    auto put = [&](int d, int stage) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            v4i x = rb[d][i];
            if constexpr (R4) { // even and odd columns, back in order
                constexpr unsigned HI = 0xF0F0F0F0u, FIRST = 0x05010400u, LAST = 0x07030602u;
                const unsigned e0 = ((unsigned)x.x << 4) & HI, o0 = (unsigned)x.x & HI, e1 = ((unsigned)x.y << 4) & HI, o1 = (unsigned)x.y & HI;
                x = (v4i){(int)__builtin_amdgcn_perm(o0, e0, FIRST), (int)__builtin_amdgcn_perm(o0, e0, LAST),
                          (int)__builtin_amdgcn_perm(o1, e1, FIRST), (int)__builtin_amdgcn_perm(o1, e1, LAST)};
            }
            *reinterpret_cast<v4i *>(lds + stage * STAGE + to[i]) = x;
        }
    };
    unsigned rd0[NT], rd1[NT]; // rows 0 .. 7 and 8 .. 15 of the lane group's block of 16
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        const unsigned base = ((kg * 4 + g) * NT + ct) * 256 + ((ii ^ (ct * (8 / NT))) * 16) + 8 * (lane & 1);
        rd0[ct] = base + (g & 1) * 128;
        rd1[ct] = base + ((g & 1) ^ 1) * 128;
    }
    v4i bop[2][NT];
    auto fetch = [&](int stage, v4i (&b)[NT]) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) { // (the kernel has no other LDS: the stages start at address 0)
            const v2i d0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(uintptr_t)(rd0[ct] + stage * STAGE));
            const v2i d1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(uintptr_t)(rd1[ct] + stage * STAGE));
            b[ct] = (v4i){d0.x, d0.y, d1.x, d1.y};
        }
    };
    v4i acc[PL][RF * NT];
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
        for (int i = 0; i < RF * NT; ++i) acc[p][i] = (v4i){0, 0, 0, 0};
    auto multiply = [&](const v4i (&b)[NT], int d, int f) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                acc[p][f * NT + ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b[ct], ra[d][f][p], acc[p][f * NT + ct], 0, 0, 0);
    };

    // ---- the product ------------------------------------------------------------------------------------------
    // The loads before the loop are in the order in which the loop issues them, so that the compiler's counted waits are the
    // loop's own.
    const int steps = (a.nch + WK - 1) / WK;
    auto load_a_all = [&](int s) {
#pragma unroll
        for (int f = 0; f < RF; ++f) load_a(s, s % AH, f);
    };
#pragma unroll
    for (int d = 0; d < AH; ++d) {
        load_b(d);
        if (d >= 3) load_a_all(d - 3);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int d = 0; d < STAGES - 1; ++d) {
        put(d, d);
        load_b(d);
        load_a_all(AH - 3 + d);
        __builtin_amdgcn_sched_barrier(0);
    }
    // (memory is fenced for the compiler only: see the loop's end)
    auto in_order = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        in_order();
    };
    mcu::lgkm_wait();
    barrier();
    fetch(0, bop[0]);
    mcu::lgkm_wait();
    barrier();
    for (int s0 = 0; s0 < steps; s0 += AH) { // (surplus steps multiply by rows of zeros)
#pragma unroll
        for (int d = 0; d < AH; ++d) {
            put((d + 3) % AH, (d + 3) % STAGES);
            in_order();                                         // (the writes are issued first: what waits for the reads has waited for them)
            fetch((d + 1) % STAGES, bop[(d + 1) & 1]);
            load_b((d + 3) % AH);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < RF; ++f) {
                multiply(bop[d & 1], d, f);
                __builtin_amdgcn_sched_barrier(0);
                load_a(s0 + d + AH, d, f);
                __builtin_amdgcn_sched_barrier(0);
            }
            // The stage that the next step overwrites held this step's rows, which every wave has consumed; the one it reads
            // was written a step before this one, ahead of that step's reads, which have returned since (LDS works in order).
            barrier();
        }
    }

    // ---- the sums of the WK groups, each of which finishes its share of the tiles ------------------------------
    if constexpr (WK > 1) {
        v4i *part = reinterpret_cast<v4i *>(lds);
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < RF * NT; ++i) part[(w * (RF * NT) + i) * 64 + lane] = acc[p][i];
            __syncthreads();
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                v4i s = part[(rw * (RF * NT) + kg * OWN + o) * 64 + lane];
#pragma unroll
                for (int k = 1; k < WK; ++k) s += part[((k * WR + rw) * (RF * NT) + kg * OWN + o) * 64 + lane];
                acc[p][o] = s;
            }
        }
    }
    // the product is rounded to fp32 before fp16: the compiler must not fold multiplication and conversion into one instruction
    auto scaled = [&](v4i s) -> v4f {
        v4f f = {s.x * a.out_scale, s.y * a.out_scale, s.z * a.out_scale, s.w * a.out_scale};
        asm("" : "+v"(f));
        return f;
    };
    const int es = a.float_out == 2 ? 2 : 4;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
        const int i = kg * OWN + o, f = i / NT, ct = i % NT;
        const int64_t row = (int64_t)((tm * WR + rw) * RF + f) * 16 + j;
        const int col = col0 + ct * 16 + 4 * g;
        // every plane's sum is exact in int32 (nibbles: after the shift); the recombination wraps
        v4i v = R4 ? acc[0][o] >> 4 : acc[0][o];
        if constexpr (PL == 2) v = (v << 8) + (R4 ? acc[1][o] >> 4 : acc[1][o]);
        if (row < a.rows && col < a.cols) {
            uint8_t *c = static_cast<uint8_t *>(a.C) + (row * a.ldc + col) * es;
            if (a.float_out == 2) __builtin_nontemporal_store(mcu::to_half4(scaled(v)), reinterpret_cast<mcu::v4h *>(c));
            else __builtin_nontemporal_store(a.float_out ? __builtin_bit_cast(v4i, scaled(v)) : v, reinterpret_cast<v4i *>(c));
        }
    }
}

template <int TILE, int PL, bool R4, int NT, int RF, int WR, int W> hipError_t launch_one(const DenseArgs &args, hipStream_t s)
{
    constexpr int AH = dense_tile_turn(TILE);
    static_assert(dense_tile_rows(TILE, PL) == 16 * RF * WR && dense_tile_cols(TILE) == 16 * NT && dense_tile_share(TILE) == W / WR, "the planner's tile");
    auto kern = spmm_dense_kernel<PL, R4, NT, RF, WR, W, AH>;
    constexpr int WK = W / WR, RING = STAGES * WK * NT * 1024, SUMS = WK > 1 ? W * RF * NT * 1024 : 0, LDS = RING > SUMS ? RING : SUMS;
    DenseArgs a = args;
    a.tm = (a.nrb + WR * RF - 1) / (WR * RF);
    a.tn = (a.cols + 16 * NT - 1) / (16 * NT);
    if (LDS > 65536) { // more than 64 KB of LDS per workgroup has to be asked for
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3((unsigned)((a.tm * a.tn + 7) / 8 * 8)), dim3(64 * W), LDS, s, a);
}

template <int PL, bool R4> hipError_t launch_tile(const DenseArgs &a, int tile, hipStream_t s)
{
    constexpr int WIDE = PL == 1 ? 2 : 1; // (see dense_tile_rows)
    switch (tile) {
    case 0: return launch_one<0, PL, R4, 8, WIDE, 8, 8>(a, s);
    case 1: return launch_one<1, PL, R4, 8, WIDE, 4, 8>(a, s);
    case 2: return launch_one<2, PL, R4, 4, 2, 4, 8>(a, s);
    case 3: return launch_one<3, PL, R4, 4, 1, 4, 8>(a, s);
    case 4: return launch_one<4, PL, R4, 4, 1, 2, 8>(a, s);
    case 5: return launch_one<5, PL, R4, 2, 1, 2, 4>(a, s);
    default: return hipErrorInvalidValue;
    }
}

// The dense copy from the panel format: a workgroup makes FILL_CHUNKS chunks of one block of 16 rows in LDS, zeros included, and
// writes them out whole.  A wave takes whole panels (two share one with V = 8) and only their slots with columns of these chunks, which
// it finds by trying 64 places at a time (columns ascend).  One byte per lane and LDS write, a slot's V rows one after the other.
// Bound by the chain columns - values - LDS.  What it adds to new values, us, against a workgroup that goes through all slots of its panels one
// panel after the other: 4096 x 4096, half empty, V = 2 17.7 -> 13.0; 2710 x 7060, 77 %, V = 2 51.6 -> 14.7; 512 x 8192, half empty, V = 4
// 19.1 -> 6.1; 2048 x 2048, V = 4, L16-R8 12.3 -> 8.5.
constexpr int FILL_CHUNKS = 16;

// the first of slots lo .. hi whose column is `col` or more (hi: none); the same in all lanes
__device__ __forceinline__ int first_slot(const int32_t *slot_idx, int lo, int hi, int col, int lane)
{
    while (lo < hi) {
        const int step = (hi - lo + 63) / 64, at = lo + lane * step;
        const int n = __popcll(__ballot(at < hi && slot_idx[at] < col));
        if (n == 0) break;
        hi = min(hi, lo + n * step);
        lo += (n - 1) * step + 1;
    }
    return lo;
}

template <int V, int BITS> __global__ __launch_bounds__(256) void dense_fill_kernel(DenseFillArgs a)
{
    constexpr int PL = BITS == 16 ? 2 : 1, PANELS = 16 / V, SHARE = PANELS < 4 ? 4 / PANELS : 1; // waves of a panel
    __shared__ __attribute__((aligned(16))) uint8_t tile[FILL_CHUNKS * PL * 1024];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int block = blockIdx.x, c0 = blockIdx.y * FILL_CHUNKS, chunks = min(FILL_CHUNKS, a.nch - c0), bytes = chunks * PL * 1024;
    for (int i = tid * 16; i < bytes; i += 256 * 16) *reinterpret_cast<v4i *>(tile + i) = (v4i){0, 0, 0, 0};
    __syncthreads();
    for (int x = w / SHARE; x < PANELS; x += 4 / SHARE) {
        const int p = block * PANELS + x;
        if (p >= a.P) break;
        const int s1 = a.panel_ptr[2 * p + 1], first = c0 * MC_CHUNK;
        const int b = first_slot(a.slot_idx, a.panel_ptr[2 * p], s1, first, lane), e = first_slot(a.slot_idx, b, s1, first + chunks * MC_CHUNK, lane);
#pragma unroll 4
        for (int s = b + w % SHARE * 64 + lane; s < e; s += SHARE * 64) {
            const int col = a.slot_idx[s] - first, g = s >> 4 & 3, j = s & 15;
            uint8_t *to = tile + (col >> 6) * (PL * 1024) + ((col >> 4 & 3) * 16 + x * V) * 16 + (col & 15);
            const uint8_t *from = a.vals + (int64_t)(s >> 6) * (8 * V * BITS) + g * (2 * V * BITS);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if constexpr (BITS == 4) { // a nibble as a byte of its value
                    const unsigned pair = from[v * 8 + (j & 7)];
                    to[v * 16] = (uint8_t)((int)(j < 8 ? pair << 28 : pair << 24) >> 28);
                } else {
#pragma unroll
                    for (int q = 0; q < PL; ++q) to[q * 1024 + v * 16] = from[q * (16 * V) + v * 16 + j];
                }
            }
        }
    }
    __syncthreads();
    uint8_t *out = a.dst + ((int64_t)block * a.nch + c0) * (PL * 1024);
    for (int i = tid * 16; i < bytes; i += 256 * 16) *reinterpret_cast<v4i *>(out + i) = *reinterpret_cast<const v4i *>(tile + i);
}

} // namespace

hipError_t launch_spmm_dense(mc_prec prec, const DenseArgs &a, int tile, hipStream_t s)
{
    if (a.nrb == 0 || a.cols == 0) return hipSuccess;
    switch (prec) {
    case MC_L8R8: return launch_tile<1, false>(a, tile, s);
    case MC_L8R4:
    case MC_L4R4: return launch_tile<1, true>(a, tile, s);
    case MC_L16R8: return launch_tile<2, false>(a, tile, s);
    case MC_L16R4:
    case MC_L12R4: return launch_tile<2, true>(a, tile, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_dense_fill(const DenseFillArgs &a, hipStream_t s)
{
    const int blocks = (a.P * a.V + 15) / 16;
    if (blocks == 0 || a.nch == 0) return hipSuccess;
    const dim3 grid((unsigned)blocks, (unsigned)((a.nch + FILL_CHUNKS - 1) / FILL_CHUNKS)), threads(256);
    switch (a.bits * 16 + a.V) {
    case 4 * 16 + 2: return launch_kernel(dense_fill_kernel<2, 4>, grid, threads, 0, s, a);
    case 4 * 16 + 4: return launch_kernel(dense_fill_kernel<4, 4>, grid, threads, 0, s, a);
    case 4 * 16 + 8: return launch_kernel(dense_fill_kernel<8, 4>, grid, threads, 0, s, a);
    case 8 * 16 + 2: return launch_kernel(dense_fill_kernel<2, 8>, grid, threads, 0, s, a);
    case 8 * 16 + 4: return launch_kernel(dense_fill_kernel<4, 8>, grid, threads, 0, s, a);
    case 8 * 16 + 8: return launch_kernel(dense_fill_kernel<8, 8>, grid, threads, 0, s, a);
    case 16 * 16 + 2: return launch_kernel(dense_fill_kernel<2, 16>, grid, threads, 0, s, a);
    case 16 * 16 + 4: return launch_kernel(dense_fill_kernel<4, 16>, grid, threads, 0, s, a);
    case 16 * 16 + 8: return launch_kernel(dense_fill_kernel<8, 16>, grid, threads, 0, s, a);
    default: return hipErrorInvalidValue;
    }
}
