// SDDMM kernels for gfx950.
//
// SDDMM (paper, Section 4.3): a workgroup owns one row panel of the mask.  The panel's
// V rows of Q are the row operand of v_mfma_i32_16x16x64_i8 and stay in registers for
// the whole panel (the paper keeps this block in shared memory for its warps); the rows
// of Kmat named by 16 consecutive mask vectors are the column operand.  Both operands
// are contiguous along the reduction dimension, so no transpose is needed
// (Section 4.3.1): lane group g = lane/16 covers bytes 64*kc + 16*g .. +15 of a row on
// both sides.  The waves of a workgroup take the panel's chunks of 64 vectors round-robin
// and never have to meet: every chunk produces its own outputs.
// Two kernels:
//   sddmm_staged_kernel rows of up to 1024 bytes (sddmm_nib32_kernel: 32 bytes of nibbles): Kmat rows are copied
//                      from global memory straight into LDS with coalesced 16-byte pieces
//                      (global_load_lds), then read as 128-bit MFMA operands; the
//                      16-byte segments are XOR-swizzled against bank conflicts.
//   sddmm_direct_kernel longer rows: each lane loads its 16 operand bytes from memory.
// int4 operands are widened in registers; int16 operands (L16-R16, Section 4.4) are split in
// registers into signed byte planes, the two Q planes stacked in the MFMA rows 0..7 / 8..15.
// The output is written in interchange (BCRS) order: V consecutive int32 per vector, or with the
// fused dequantisation of Section 5.3 V consecutive fp32 / fp16 values.
#include "internal.h"
#include "lds_async.h"
#include "sddmm_tile.h"

namespace {

using namespace mcs;


// four fp32 values rounded to fp16 (to nearest even; beyond the fp16 range: infinity)
__device__ __forceinline__ v4h to_half4(v4f f) { return (v4h){(_Float16)f.x, (_Float16)f.y, (_Float16)f.z, (_Float16)f.w}; }

// The workgroup's share: first slot, vectors, panel, first output vector.  COMPUTED: worked out where all panels are equally long, which saves the one
// of a wave's three dependent trips to memory that comes before its indices and rows of Q.  SCALAR: read through the scalar cache; the compiler reads
// through the vector caches once a volatile statement comes before (request_arguments), and merged with what is worked out the values stay in vector registers: four
// to nine more of them, a wave less per SIMD in nine of the kernels with float results.
// Which kernels do which is measured, three operands in turn replayed from a graph, as before either / worked out or read through the vector caches / now:
//   staged (both): 4096 x 4096, 90 % empty, Kd = 256 5.67 / 5.46 / 5.51 us, fp32 6.15 / 5.98 / 5.97; unequal panels 6.37 / 6.30 / 6.38; L16-R16, 2000 x 3100, V = 4,
//     Kd = 200, unequal 8.95 / 8.91 / 8.91
//   nib32 (scalar): 4096 x 4096, 90 %, unsigned, fp32 5.01 / 5.23 / 4.99; int32, unequal panels 4.46 / 4.57 / 4.49
//   direct, 2048 x 2048: 16 bits (both), Kd = 640, 90 % 31.5 / 31.0 / 30.8; bytes with float results (both), Kd = 1040, 80 % 42.5 / 41.6 / 41.6; with int32 results
//     (scalar) 42.0 / 42.9 / 42.05; nibbles (neither), Kd = 2112, 90 % 29.5 / 29.7 / 29.5, fp16 30.0 / 31.5 / 30.0 (scalar alone 29.95, both 31.2 and 30.3)
//   unsigned (both), bytes, 2048 x 2048, 90 %, Kd = 1040 33.0 / 31.9 / 32.0
template <bool COMPUTED, bool SCALAR> __device__ __forceinline__ v4i share_of(const SddmmArgs &a)
{
    const int p = (int)blockIdx.x, n = COMPUTED ? a.uniform_vectors : 0;
    if (COMPUTED && n > 0) return (v4i){p * ((n + MC_CHUNK - 1) / MC_CHUNK * MC_CHUNK), n, p, p * n};
    if constexpr (SCALAR) return *(__attribute__((address_space(4))) const v4i *)(uintptr_t)(a.shares + 4 * p);
    else return *reinterpret_cast<const v4i *>(a.shares + 4 * p);
}

// DQ: fused dequantisation (Section 5.3).  A compile-time switch: the integer path keeps its
// straight-line stores, which the scheduler interleaves with the next tile's MFMAs.
// float_out 3 (only with DQ): the scores leave as integer codes clamp(rint(score * out_scale)) of 8 or 16 bits,
// written into the device panel format of a sparse operand with the mask's pattern (Section 4.3: the
// SDDMM writes the format the following SpMM reads); padded slots receive zeros.  s0: first slot of the panel.
template <bool DQ>
__device__ __forceinline__ void store_scores(const SddmmArgs &a, int64_t out0, int s0, int slot, int n, int g, v4i acc)
{
    if (DQ && a.float_out == 3) {
        if (4 * g >= a.V) return;
        const int64_t gs = (int64_t)s0 + slot;                 // slot of the whole matrix
        const int sub = (int)(gs % MC_CHUNK) / 16, b = (int)(gs % 16);
        const float qmax = (a.code_bits == 16) ? 32639.f : 127.f;
        uint8_t *chunk = a.dev_vals + (int64_t)blockIdx.y * a.dev_batch_stride + (gs / MC_CHUNK) * (MC_CHUNK * a.V * a.code_bits / 8);
        const int nr = a.V - 4 * g < 4 ? a.V - 4 * g : 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r >= nr) break;
            // one fp32 product, rounded to nearest even, then clamped: the same arithmetic as the oracle's
            const float x = __builtin_rintf((float)acc[r] * a.out_scale);
            const int code = (slot < n) ? (int)__builtin_fminf(__builtin_fmaxf(x, -qmax), qmax) : 0;
            const int v = 4 * g + r;
            if (a.code_bits == 8) {
                chunk[sub * (16 * a.V) + v * 16 + b] = (uint8_t)code;
            } else {
                const int hi = (code + 128) >> 8, lo = code - hi * 256;   // two signed bytes: code = 256 * hi + lo
                chunk[sub * (32 * a.V) + v * 16 + b] = (uint8_t)hi;
                chunk[sub * (32 * a.V) + 16 * a.V + v * 16 + b] = (uint8_t)lo;
            }
        }
        return;
    }
    // accumulator register r of lane (j, g) is row 4g + r of vector `slot`
    if (slot < n && 4 * g < a.V) {
        const int64_t off = out0 + (int64_t)slot * a.V + 4 * g;
        if (!DQ) {
            int32_t *o = static_cast<int32_t *>(a.S) + off;
            if (a.V >= 4) __builtin_nontemporal_store(acc, reinterpret_cast<v4i *>(o));
            else __builtin_nontemporal_store((v2i){acc.x, acc.y}, reinterpret_cast<v2i *>(o));
        } else {
            const v4f f = {acc.x * a.out_scale, acc.y * a.out_scale, acc.z * a.out_scale, acc.w * a.out_scale};
            if (a.float_out == 1) {
                float *o = static_cast<float *>(a.S) + off;
                if (a.V >= 4) __builtin_nontemporal_store(f, reinterpret_cast<v4f *>(o));
                else { o[0] = f.x; o[1] = f.y; }
            } else {
                _Float16 *o = static_cast<_Float16 *>(a.S) + off;
                const v4h h = to_half4(f);
                if (a.V >= 4) __builtin_nontemporal_store(h, reinterpret_cast<v4h *>(o));
                else *reinterpret_cast<v2h *>(o) = (v2h){h.x, h.y};
            }
        }
    }
}


// Two int16 operands: the tile's accumulators hold Qh.Kh (rows 0 .. 7) and Ql.Kh (rows 8 .. 15, 32 lanes further up) in acc, the same with
// Kl in acc2; S = (QhKh << 16) + ((QhKl + QlKh) << 8) + QlKl.  Each half of the wave adds up the two terms that it has after one
// exchange of halves (lower lanes those of acc, upper lanes those of acc2), a second exchange brings the halves' sums together and leaves
// lane (j, g) rows 4 (g & 1) + 2 (g >> 1) and the next of vector j: every lane has a pair of rows to store.  Of two tiles the exchange
// leaves four rows of one in the lower and of the other in the upper half.
__device__ __forceinline__ v4i halves16(v4i acc, v4i acc2, int lower_shift)
{
    v4i z;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const auto s = __builtin_amdgcn_permlane32_swap((unsigned)acc[r], (unsigned)acc2[r], false, false);
        z[r] = (int)(((s[0] << 8) + s[1]) << lower_shift);   // lower: QhKh << 16 + QlKh << 8; upper: QhKl << 8 + QlKl
    }
    return z;
}
__device__ __forceinline__ v4i two_tiles(v4i z, v4i y)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const auto s = __builtin_amdgcn_permlane32_swap((unsigned)z[r], (unsigned)y[r], false, false);
        z[r] = (int)(s[0] + s[1]);
    }
    return z;
}
__device__ __forceinline__ v2i combine16(v4i acc, v4i acc2, int lower_shift)
{
    const v4i z = halves16(acc, acc2, lower_shift);
    v2i out;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const auto s = __builtin_amdgcn_permlane32_swap((unsigned)z[r], (unsigned)z[r + 2], false, false);
        out[r] = (int)(s[0] + s[1]);
    }
    return out;
}

// store_scores for the pair of rows that combine16 leaves in a lane
template <bool DQ>
__device__ __forceinline__ void store_pair(const SddmmArgs &a, int64_t out0, int s0, int slot, int n, int g, v2i s)
{
    const int row = 4 * (g & 1) + 2 * (g >> 1);
    if (DQ && a.float_out == 3) {
        if (row >= a.V) return;
        const int64_t gs = (int64_t)s0 + slot;
        const int sub = (int)(gs % MC_CHUNK) / 16, b = (int)(gs % 16);
        const float qmax = (a.code_bits == 16) ? 32639.f : 127.f;
        uint8_t *chunk = a.dev_vals + (int64_t)blockIdx.y * a.dev_batch_stride + (gs / MC_CHUNK) * (MC_CHUNK * a.V * a.code_bits / 8);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float x = __builtin_rintf((float)s[r] * a.out_scale);
            const int code = (slot < n) ? (int)__builtin_fminf(__builtin_fmaxf(x, -qmax), qmax) : 0;
            if (a.code_bits == 8) {
                chunk[sub * (16 * a.V) + (row + r) * 16 + b] = (uint8_t)code;
            } else {
                const int hi = (code + 128) >> 8, lo = code - hi * 256;
                chunk[sub * (32 * a.V) + (row + r) * 16 + b] = (uint8_t)hi;
                chunk[sub * (32 * a.V) + 16 * a.V + (row + r) * 16 + b] = (uint8_t)lo;
            }
        }
        return;
    }
    if (slot < n && row < a.V) {
        const int64_t off = out0 + (int64_t)slot * a.V + row;
        if (!DQ) {
            __builtin_nontemporal_store(s, reinterpret_cast<v2i *>(static_cast<int32_t *>(a.S) + off));
        } else {
            const float f0 = s.x * a.out_scale, f1 = s.y * a.out_scale;
            if (a.float_out == 1) {
                float *o = static_cast<float *>(a.S) + off;
                o[0] = f0; o[1] = f1;
            } else {
                const v4h h = to_half4((v4f){f0, f1, 0.f, 0.f});
                *reinterpret_cast<v2h *>(static_cast<_Float16 *>(a.S) + off) = (v2h){h.x, h.y};
            }
        }
    }
}

// LPR: 16-byte pieces (lanes) of a staged Kmat row: 4, 8, 16, 32 or 64; a row has at most that many and is always
// fetched whole.  Pieces beyond its end are fetched from its start instead (a line that is on its way anyway), and the Q
// operand is zero there, so they add nothing.
// U: 8- or 4-bit operands of which one or both are read as non-negative values (Section 4.4.1); the
// scheme is the one described at sddmm_unsigned_kernel below, here on rows staged in LDS.
//
// The unit of work of a wave is 8 KB of rows: 64 vectors of up to 128 bytes, 32 of 256, 16 of 512 (4 KB for rows of 64
// bytes, 16 KB for 1024).  What bounds the kernel on large masks is the number of 128-byte lines the gather asks L2 for
// (about 3 clocks per line and compute unit), so a row is read in one go by neighbouring lanes: cut into pieces of 128 or
// 256 bytes, a row that is not aligned to lines costs one more line per piece.  On small masks it is the chain row
// numbers -> rows -> MFMA -> stores.  A unit's rows are copied straight into the wave's one stage of LDS; its operands
// are then taken into registers, which frees the stage for the next unit's rows while the MFMAs and stores of this one
// run (a second stage would halve the waves of a compute unit, staging through registers costs LDS writes: 2 - 8 % slower).
// L8-R8, 4096 x 4096, V = 8, 90 % sparse, Kd = 256: 6.2 -> 5.9 us; 1224 x 7932, V = 4, 80 %, Kd = 464 58.7 -> 21.7 us, L16-R16,
// 2000 x 3100, V = 4, 90 %, Kd = 200 13.6 -> 8.6 us (row lengths that the direct kernel used to take: there the lanes that read
// one row are 16 apart and their requests are not combined, 9 TB/s of rows from L2 against 25 coalesced).
// With int16 operands it is the instructions, too (the same rows as int8: 6.9 us where int16 took 8.9, equal panels): Kmat's bytes
// are taken apart without a carry, halves of the wave combine a tile's four sums by two exchanges in registers, and offsets are 32
// bits wide where they can be: 8.9 -> 7.9; with rows above 512 bytes (5760 x 2546, V = 8, 71 %, Kd = 280) 43.6 -> 32.7.
// Loads and stores take a compute unit 16 clocks where a lane has 8 or 16 bytes, also where half of the lanes have nothing, and 4.6
// where it has 4: the indices are shared by the lanes of a row, and where a unit has several tiles two of them are stored at once.  54 drawn masks, three
// operands in turn from a graph, 1.027x in the mean (4096 x 4096, 90 % sparse, Kd = 256 5.9 -> 5.6 us; 758 x 5997, V = 2, Kd = 128 13.2 -> 11.4; L16-R16,
// 4360 x 6043, V = 8, Kd = 72 31.5 -> 28.7); 16-bit ones of 3 us 1 % slower.
// SHORT: Kmat spans less than 4 GiB, its rows and their length fit 24 bits.
template <int PB, int LPR, bool DQ, bool U, bool SHORT>
__global__ __launch_bounds__(512) void sddmm_staged_kernel(SddmmArgs a)
{
    mcu::request_arguments(a);
    constexpr int RB = LPR * 16, NI = (LPR == 4) ? 4 : (LPR == 64 ? 16 : 8), RPI = 64 / LPR, UNIT = NI * RPI, TILES = UNIT / 16;
    constexpr int KC = RB / StepBytes<PB>::value;
    constexpr int SW = (LPR < 16) ? LPR : 16;       // pieces of a row that the swizzle permutes
    static_assert(KC >= 1, "a row must fill at least one MFMA step");
    static_assert(!U || PB == 8 || PB == 4, "unsigned operands: 4 and 8 bits");
    constexpr int QR = (U && PB == 4) ? 2 : 1; // registers per step of the Q operand (unsigned nibbles are widened once, up front)
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int rg = lane / LPR, seg = lane % LPR;
    const int batch = blockIdx.y;
    const v4i share = share_of<true, true>(a);
    const int s0 = share.x, n = share.y, panel = share.z;
    // (codes written into an operand's device format also cover the padded slots, with zeros)
    const int n_all = (DQ && a.float_out == 3) ? (n + MC_CHUNK - 1) / MC_CHUNK * MC_CHUNK : n;
    const int nunits = (n_all + UNIT - 1) / UNIT;
    const int nmy = (nunits > w) ? (nunits - w + nw - 1) / nw : 0;
    if (nmy == 0) return;
    // piece i of a unit: lane (rg, seg) fetches piece seg of the row in slot rg*NI + i.  The lanes of a row need the same indices: each of
    // four neighbours loads every fourth one, and copy i takes its index from neighbour i % 4.  (A load of 4 bytes a lane takes a compute
    // unit 4.6 clocks, one of 16 as long as a copy of 1 KB, 16: loaded whole by every lane, the indices were up to a quarter of the copies.)
    constexpr int NX = NI / 4;
    const int32_t *idx = a.slot_idx + s0 + rg * NI + (lane & 3);
    int ixn[NX];
    auto load_idx = [&](int u) {
#pragma unroll
        for (int t = 0; t < NX; ++t) ixn[t] = idx[u * UNIT + 4 * t];
    };
    auto from_neighbour = [&](auto I, int x) -> int { // (with all lanes active)
        return __builtin_amdgcn_mov_dpp(x, decltype(I)::value % 4 * 0x55, 0xF, 0xF, true); // quad_perm [q,q,q,q]
    };
    load_idx(w);
    const int64_t out0 = (int64_t)batch * a.S_batch_stride + (int64_t)share.w * a.V;
    const uint8_t *Km = a.Kmat + (int64_t)batch * a.K_batch_stride;

    v4i qf[KC * QR];
    const uint8_t *Qpanel = a.Q + (int64_t)batch * a.Q_batch_stride + (int64_t)panel * a.V * a.ldq_bytes;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const v4i nib = {NIBBLE_HI, NIBBLE_HI, NIBBLE_HI, NIBBLE_HI};
    int qx1 = (U && a.lhs_unsigned) ? (int)0x80808080 : 0, kx1 = (U && a.rhs_unsigned) ? (int)0x80808080 : 0;
    if (U) asm("" : "+v"(qx1), "+v"(kx1));
    const v4i qx = {qx1, qx1, qx1, qx1}, kx = {kx1, kx1, kx1, kx1};
    v4i raw_q[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) raw_q[kc] = load_q<PB>(Qpanel, a.ldq_bytes, a.V, a.row_bytes, kc, j, g);

    // LDS: the row of slot s at byte (s % NI) * 1024 + (s / NI) * RB, its piece p at position p ^ swz(s): the 16 rows of a
    // tile, read at one piece number by 16 lanes, spread over all banks
    char *stage = lds + w * (UNIT * RB);
    const unsigned stage_u = mcu::lds_addr_uniform(stage);
    auto swz = [](int s) { return LPR < 16 ? (s ^ (s >> 3)) & (SW - 1) : s & 15; };
    int off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int p = seg ^ swz(rg * NI + i);
        off[i] = p * 16 < a.row_bytes ? p * 16 : 0;
    }
    auto request = [&]() {
        unsigned to = stage_u;
        if (U && LPR == 64) asm("" : "+s"(to)); // (sixteen places kept in scalar registers would be spilled)
        if constexpr (SHORT) { // (multiplied by the lane that holds an index, handed over in the sum)
            int at[NX];
#pragma unroll
            for (int t = 0; t < NX; ++t) at[t] = (int)__umul24((unsigned)ixn[t], (unsigned)a.ldk_bytes);
            mcu::static_for<NI>([&](auto I) {
                constexpr int i = decltype(I)::value;
                mcu::copy16_to_lds(Km, (unsigned)from_neighbour(I, at[i / 4]) + (unsigned)off[i], to + i * 1024);
            });
        } else {
            mcu::static_for<NI>([&](auto I) {
                constexpr int i = decltype(I)::value;
                mcu::copy16_to_lds(Km + ((int64_t)from_neighbour(I, ixn[i / 4]) * a.ldk_bytes + off[i]), to + i * 1024);
            });
        }
    };
    request();
    if (nmy > 1) load_idx(w + nw);

    // sum over the reduction of the Q operand bytes, of rows 4g .. 4g+3 (U, and int16)
    v4i rq = {0, 0, 0, 0};
    const int lower_shift = lane < 32 ? 8 : 0;
    int ones8 = (j == 8) ? 0x01010101 : 0, of_panel = (j < a.V) ? -1 : 0;
    asm("" : "+v"(ones8), "+v"(of_panel));
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        if (!U) {
            qf[kc] = raw_q[kc];
            if (PB == 16) rq = __builtin_amdgcn_mfma_i32_16x16x64_i8(raw_q[kc], ones, rq, 0, 0, 0);
        } else {
            // rows of the panel: the operand bytes; MFMA row 8: all ones (it collects the sums of the Kmat
            // operand bytes of every output column); other rows, and everything beyond the row end: zero
            // (bit masks in vector registers: as conditions they would take two scalar registers per step)
            int row1 = (kc * 64 + g * 16 - a.row_bytes) >> 31;
            asm("" : "+v"(row1));
            const int keep1 = row1 & of_panel, one1 = row1 & ones8;
            const v4i keep = {keep1, keep1, keep1, keep1}, one = {one1, one1, one1, one1};
#pragma unroll
            for (int t = 0; t < QR; ++t) {
                const v4i q = (((PB == 8) ? (raw_q[kc] ^ qx) : (((t == 0 ? (raw_q[kc] << 4) : raw_q[kc]) & nib) ^ qx)) & keep) | one;
                qf[kc * QR + t] = q;
                rq = __builtin_amdgcn_mfma_i32_16x16x64_i8(q, ones, rq, 0, 0, 0);
            }
        }
    }
    const int nred = a.row_bytes * (PB == 4 ? 2 : 1);                    // reduction elements
    int cqck = (U && a.lhs_unsigned && a.rhs_unsigned) ? (PB == 4 ? 64 : 16384) * nred : 0;
    if (U) asm("" : "+v"(cqck)); // (scalar registers are scarce here)

    for (int k = 0; k < nmy; ++k) {
        const int u = w + k * nw;
        // This unit's rows have landed.  (Integer outputs: the stores of the unit before, one for two tiles or for one, were issued after this
        // unit's copies -- only the last unit can have tiles without a store -- and need not be waited for.)
        constexpr bool IN_TWOS = !U && TILES > 1;
        constexpr int STORES = IN_TWOS ? TILES / 2 : TILES;
        if (k == 0 || DQ) mcu::vm_wait<0>();
        else mcu::vm_wait<STORES>();
        // The operands of the whole unit first, so that the stage is free for the next unit's rows before the MFMAs (rows
        // of 1024 bytes: their operands are more than the registers hold, they are read one by one).
        constexpr int OPS = (PB == 16) ? 2 * KC : KC;
        constexpr bool EARLY = LPR < 64;
        v4i kt[TILES][OPS];
        auto read_op = [&](int tl, int kc) -> v4i {
            const int s = tl * 16 + j, i = s % NI;
            const char *rowp = stage + i * 1024 + (s / NI) * RB;
            const int p = (PB == 16) ? (kc >> 1) * 8 + 2 * g + (kc & 1) : kc * 4 + g;
            return *reinterpret_cast<const v4i *>(rowp + (p ^ swz(s)) * 16);
        };
        auto next_unit = [&]() {
            mcu::lgkm_wait();                       // the reads have returned: the stage may be overwritten
            if (k + 1 < nmy) {
                request();
                if (k + 2 < nmy) load_idx(u + 2 * nw);
            }
        };
        if (EARLY) {
#pragma unroll
            for (int tl = 0; tl < TILES; ++tl)
#pragma unroll
                for (int kc = 0; kc < OPS; ++kc) kt[tl][kc] = read_op(tl, kc);
            next_unit();
        }
        v4i even = {0, 0, 0, 0};
#pragma unroll
        for (int tl = 0; tl < TILES; ++tl) {
            // (int16: the low bytes of Kmat enter as u - 128, and 128 times the sum of Q goes in here)
            v4i acc = {0, 0, 0, 0}, acc2 = (PB == 16) ? rq << 7 : (v4i){0, 0, 0, 0};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                if (PB == 16) {
                    v4i kh, kl;
                    if (EARLY) bytes16(kt[tl][2 * kc], kt[tl][2 * kc + 1], kh, kl);
                    else bytes16(read_op(tl, 2 * kc), read_op(tl, 2 * kc + 1), kh, kl);
                    mma_step<PB>(qf[kc], kh, kl, acc, acc2);
                } else {
                    const v4i kf = EARLY ? kt[tl][kc] : read_op(tl, kc);
                    if (!U) {
                        mma_step<PB>(qf[kc], kf, kf, acc, acc2);
                    } else if (PB == 8) {
                        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qf[kc], kf ^ kx, acc, 0, 0, 0);
                    } else {
                        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qf[kc * 2], ((kf << 4) & nib) ^ kx, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qf[kc * 2 + 1], (kf & nib) ^ kx, acc, 0, 0, 0);
                    }
                }
            }
            if (!EARLY) next_unit();                // (a unit of these is one tile)
            const int slot = u * UNIT + tl * 16 + j;
            if (IN_TWOS) {
                // two tiles' rows 0 .. 7 side by side, so that all lanes have four rows to store: a store takes a compute unit as long for half the lanes
                const v4i z = PB == 16 ? halves16(acc, acc2, lower_shift) : finish_tile<PB>(acc, acc2);
                if (tl % 2 == 0) {
                    even = z;
                } else {
                    v4i both;
                    if (PB == 16) {
                        both = two_tiles(even, z);
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) both[r] = (int)__builtin_amdgcn_permlane32_swap((unsigned)even[r], (unsigned)z[r], false, false)[0];
                    }
                    store_scores<DQ>(a, out0, s0, slot - 16 + 16 * (g >> 1), n, g & 1, both);
                }
            } else if (PB == 16) {
                store_pair<DQ>(a, out0, s0, slot, n, g, combine16(acc, acc2, lower_shift));
            } else if (!U) {
                store_scores<DQ>(a, out0, s0, slot, n, g, finish_tile<PB>(acc, acc2));
            } else {
                // sum (q'+cq)(k'+ck) = sum q'k' + ck sum q' + cq sum k' + cq ck n, with cq = ck = 128 in the
                // scale the operand bytes carry (nibbles: 16 x their value)
                const int cs = __shfl(acc[0], 32 + j); // MFMA row 8 (lane group 2, register 0) of this lane's column
                if (a.rhs_unsigned) acc += rq << 7;
                if (a.lhs_unsigned) acc += (v4i){cs << 7, cs << 7, cs << 7, cs << 7};
                if (PB == 4) acc = acc >> 8;
                acc += (v4i){cqck, cqck, cqck, cqck};
                store_scores<DQ>(a, out0, s0, slot, n, g, acc);
            }
        }
    }
}

// Rows of 32 bytes of packed nibbles (Kd = 64 with 4-bit operands): one MFMA step per tile.  The 64
// reduction elements of a row fill the step exactly when lane groups 0 and 1 take the even elements
// of the two 16-byte pieces (low nibbles, shifted up) and groups 2 and 3 the odd ones (high nibbles),
// on both operand sides: sums do not depend on the order of their terms.  Both operands carry a
// factor 16.  Staging as in sddmm_staged_kernel: copy instruction i (of 2) brings the rows of the
// slots 2*rg + i, rg = lane / 2, into LDS rows i*32 + rg, pieces XOR-swizzled with i.
template <int WK, bool DQ, bool U>
__global__ __launch_bounds__(64 * WK) void sddmm_nib32_kernel(SddmmArgs a)
{
    mcu::request_arguments(a);
    constexpr int RB = 32;
    __shared__ __attribute__((aligned(16))) char lds[WK * 64 * RB];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int rg = lane >> 1, seg = lane & 1;
    const int batch = blockIdx.y;
    const v4i share = share_of<false, true>(a);
    const int s0 = share.x, n = share.y, panel = share.z;
    const int nch = (n + MC_CHUNK - 1) / MC_CHUNK;
    const int32_t *idx = a.slot_idx + s0;
    const int64_t out0 = (int64_t)batch * a.S_batch_stride + (int64_t)share.w * a.V;
    const uint8_t *Km = a.Kmat + (int64_t)batch * a.K_batch_stride;
    char *stage = lds + w * (64 * RB);

    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const v4i nib = {NIBBLE_HI, NIBBLE_HI, NIBBLE_HI, NIBBLE_HI};
    const int qx1 = (U && a.lhs_unsigned) ? (int)0x80808080 : 0, kx1 = (U && a.rhs_unsigned) ? (int)0x80808080 : 0;
    const v4i qx = {qx1, qx1, qx1, qx1}, kx = {kx1, kx1, kx1, kx1};
    // this lane's operand from 16 raw bytes: even elements (groups 0, 1) or odd elements (groups 2, 3)
    auto widen = [&](v4i raw) -> v4i { return ((g < 2) ? (raw << 4) : raw) & nib; };

    v4i qop = {0, 0, 0, 0};
    if (j < a.V) {
        const uint8_t *qrow = a.Q + (int64_t)batch * a.Q_batch_stride + (int64_t)(panel * a.V + j) * a.ldq_bytes;
        qop = widen(*reinterpret_cast<const v4i *>(qrow + (g & 1) * 16)) ^ qx;
    } else if (U && j == 8) {
        qop = ones; // MFMA row 8 collects the sums of the Kmat operand bytes of every output column
    }
    v4i rq = {0, 0, 0, 0}; // U: rows 4g .. 4g+3: sum over the reduction of the Q operand bytes
    if (U) rq = __builtin_amdgcn_mfma_i32_16x16x64_i8(qop, ones, rq, 0, 0, 0);
    const int cqck = (U && a.lhs_unsigned && a.rhs_unsigned) ? 64 * 64 : 0; // cq * ck per element, 64 elements

    const int nmy = (nch > w) ? (nch - w + WK - 1) / WK : 0;
    v2i idxv = {0, 0};
    if (nmy > 0) idxv = *reinterpret_cast<const v2i *>(idx + w * MC_CHUNK + rg * 2);
    for (int k = 0; k < nmy; ++k) {
        const int c = w + k * WK;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t *)(Km + (int64_t)idxv[i] * a.ldk_bytes + ((seg ^ i) * 16)),
                                             (lptr_t *)(stage + i * 1024), 16, 0, 0);
        if (k + 1 < nmy) {
            idxv = *reinterpret_cast<const v2i *>(idx + (c + WK) * MC_CHUNK + rg * 2);
            asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); // rows landed, indices may still fly
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
#pragma unroll
        for (int tl = 0; tl < 4; ++tl) {
            const int s = tl * 16 + j;              // slot within the chunk
            const int i = s & 1, r = s >> 1;        // its copy instruction and row group
            const v4i kf = *reinterpret_cast<const v4i *>(stage + i * 1024 + r * RB + (((g & 1) ^ i) * 16));
            v4i acc = {0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qop, widen(kf) ^ kx, acc, 0, 0, 0);
            if (U) {
                const int cs = __shfl(acc[0], 32 + j); // MFMA row 8 (lane group 2, register 0) of this lane's column
                if (a.rhs_unsigned) acc += rq << 7;
                if (a.lhs_unsigned) acc += (v4i){cs << 7, cs << 7, cs << 7, cs << 7};
            }
            acc = acc >> 8; // both operands carried a factor 16
            if (U) acc += (v4i){cqck, cqck, cqck, cqck};
            store_scores<DQ>(a, out0, s0, c * MC_CHUNK + s, n, g, acc);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // reads done before the rows are overwritten
    }
}

// KC = number of MFMA steps along a row kept in registers (0: any length, Q re-read).
template <int PB, int KC, bool DQ>
__global__ __launch_bounds__(64 * SDDMM_WAVES) void sddmm_direct_kernel(SddmmArgs a)
{
    // (Not for bytes: 512 x 2048, V = 2, 80 % empty, Kd = 1040 took 25.5 us as fp16 with it, 24.5 without; 4-bit rows 1.04x as long without.)
    if constexpr (PB != 8) mcu::request_arguments(a);
    constexpr int STEP = StepBytes<PB>::value, LANEB = STEP / 4; // bytes per step / per lane and step
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int batch = blockIdx.y;
    const v4i share = share_of<PB == 16 || (PB == 8 && DQ), PB != 4>(a);
    const int s0 = share.x, n = share.y, panel = share.z;
    // (codes written into an operand's device format also cover the padded slots of the last chunk, with zeros)
    const int ntile = (DQ && a.float_out == 3) ? (n + MC_CHUNK - 1) / MC_CHUNK * 4 : (n + 15) / 16;
    const int64_t out0 = (int64_t)batch * a.S_batch_stride + (int64_t)share.w * a.V;
    const uint8_t *Qpanel = a.Q + (int64_t)batch * a.Q_batch_stride + (int64_t)panel * a.V * a.ldq_bytes;
    const uint8_t *Km = a.Kmat + (int64_t)batch * a.K_batch_stride + g * LANEB;
    const int kc_n = (a.row_bytes + STEP - 1) / STEP;

    // this lane's piece of step kc of a Kmat row: (k, k2) = the operand (8 / 4 bit) or its planes
    auto load_k = [&](const uint8_t *kr, int kc, v4i &k, v4i &k2) {
        k = k2 = (v4i){0, 0, 0, 0};
        const int off = kc * STEP + g * LANEB;
        if (off < a.row_bytes) {
            const v4i x = *reinterpret_cast<const v4i *>(kr + kc * STEP);
            if (PB == 16) {
                v4i y = {0, 0, 0, 0};
                if (off + 16 < a.row_bytes) y = *reinterpret_cast<const v4i *>(kr + kc * STEP + 16);
                split16(x, y, k, k2);
            } else {
                k = x;
            }
        }
    };

    v4i qf[KC > 0 ? KC : 1];
    if (KC > 0) {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) qf[kc] = load_q<PB>(Qpanel, a.ldq_bytes, a.V, a.row_bytes, kc, j, g);
    }

    for (int t = w; t < ntile; t += SDDMM_WAVES) {
        const int slot = t * 16 + j;
        const int row = a.slot_idx[s0 + slot]; // padded slots name a valid row
        const uint8_t *kr = Km + (int64_t)row * a.ldk_bytes;
        v4i acc = {0, 0, 0, 0}, acc2 = {0, 0, 0, 0};
        if (KC > 0) {
            v4i kf[KC > 0 ? KC : 1], kf2[KC > 0 ? KC : 1];
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) load_k(kr, kc, kf[kc], kf2[kc]);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) mma_step<PB>(qf[kc], kf[kc], kf2[kc], acc, acc2);
        } else {
            for (int kc = 0; kc < kc_n; ++kc) {
                v4i k, k2;
                load_k(kr, kc, k, k2);
                const v4i q = load_q<PB>(Qpanel, a.ldq_bytes, a.V, a.row_bytes, kc, j, g);
                mma_step<PB>(q, k, k2, acc, acc2);
            }
        }
        store_scores<DQ>(a, out0, s0, slot, n, g, finish_tile<PB>(acc, acc2));
    }
}

// ---- unsigned 8- and 4-bit operands (Section 4.4.1), any row length ---------------------------
// The signed MFMA takes an unsigned value u as u - c (c = 128, or 8 for a nibble: one XOR of the
// top bit of the operand byte); sum (q'+cq)(k'+ck) = sum q'k' + ck sum q' + cq sum k' + cq ck n.
// sum q' per Q row comes from an MFMA against an all-ones column operand (once per wave), sum k'
// per gathered Kmat row from MFMA row 8, which is free (V <= 8) and is fed an all-ones row operand.
// Reduction bytes beyond the row end are zero on both sides before the XOR, so they take part in
// every term consistently and n counts them.
template <int PB, bool DQ>
__global__ __launch_bounds__(64 * SDDMM_WAVES) void sddmm_unsigned_kernel(SddmmArgs a)
{
    static_assert(PB == 8 || PB == 4, "unsigned operands: 4 and 8 bits");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int batch = blockIdx.y;
    const v4i share = share_of<true, true>(a);
    const int s0 = share.x, n = share.y, panel = share.z;
    // (codes written into an operand's device format also cover the padded slots of the last chunk, with zeros)
    const int ntile = (DQ && a.float_out == 3) ? (n + MC_CHUNK - 1) / MC_CHUNK * 4 : (n + 15) / 16;
    const int64_t out0 = (int64_t)batch * a.S_batch_stride + (int64_t)share.w * a.V;
    const uint8_t *Qrow = a.Q + (int64_t)batch * a.Q_batch_stride + (int64_t)(panel * a.V + (j < a.V ? j : 0)) * a.ldq_bytes + g * 16;
    const uint8_t *Km = a.Kmat + (int64_t)batch * a.K_batch_stride + g * 16;
    const int kc_n = (a.row_bytes + 63) / 64;
    const int qx = a.lhs_unsigned ? (int)0x80808080 : 0, kx = a.rhs_unsigned ? (int)0x80808080 : 0;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const v4i nib = {NIBBLE_HI, NIBBLE_HI, NIBBLE_HI, NIBBLE_HI};

    // operands of step kc: (q0, q1) row operands and (k0, k1) column operands; 8 bit uses the first of each
    auto q_ops = [&](int kc, v4i &q0, v4i &q1) {
        v4i raw = {0, 0, 0, 0};
        if (kc * 64 + g * 16 < a.row_bytes) raw = *reinterpret_cast<const v4i *>(Qrow + kc * 64);
        const v4i x = {qx, qx, qx, qx};
        if (PB == 8) { q0 = raw ^ x; q1 = q0; }
        else { q0 = ((raw << 4) & nib) ^ x; q1 = (raw & nib) ^ x; }
        if (j >= a.V) q0 = q1 = (j == 8) ? ones : (v4i){0, 0, 0, 0};
    };
    auto k_ops = [&](const uint8_t *kr, int kc, v4i &k0, v4i &k1) {
        v4i raw = {0, 0, 0, 0};
        if (kc * 64 + g * 16 < a.row_bytes) raw = *reinterpret_cast<const v4i *>(kr + kc * 64);
        const v4i x = {kx, kx, kx, kx};
        if (PB == 8) { k0 = raw ^ x; k1 = k0; }
        else { k0 = ((raw << 4) & nib) ^ x; k1 = (raw & nib) ^ x; }
    };

    v4i rq = {0, 0, 0, 0}; // rows 4g .. 4g+3: sum over the reduction of the Q operand bytes
    for (int kc = 0; kc < kc_n; ++kc) {
        v4i q0, q1;
        q_ops(kc, q0, q1);
        rq = __builtin_amdgcn_mfma_i32_16x16x64_i8(q0, ones, rq, 0, 0, 0);
        if (PB == 4) rq = __builtin_amdgcn_mfma_i32_16x16x64_i8(q1, ones, rq, 0, 0, 0);
    }
    const int nred = kc_n * (PB == 4 ? 128 : 64);                       // reduction elements, padding included
    const int cqck = (a.lhs_unsigned && a.rhs_unsigned) ? (PB == 4 ? 64 : 16384) * nred : 0;

    for (int t = w; t < ntile; t += SDDMM_WAVES) {
        const int slot = t * 16 + j;
        const int row = a.slot_idx[s0 + slot]; // padded slots name a valid row
        const uint8_t *kr = Km + (int64_t)row * a.ldk_bytes;
        v4i acc = {0, 0, 0, 0};
        for (int kc = 0; kc < kc_n; ++kc) {
            v4i q0, q1, k0, k1;
            q_ops(kc, q0, q1);
            k_ops(kr, kc, k0, k1);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(q0, k0, acc, 0, 0, 0);
            if (PB == 4) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(q1, k1, acc, 0, 0, 0);
        }
        const int cs = __shfl(acc[0], 32 + j); // MFMA row 8 (lane group 2, register 0) of this lane's column
        if (a.rhs_unsigned) acc += rq << 7;
        if (a.lhs_unsigned) acc += (v4i){cs << 7, cs << 7, cs << 7, cs << 7};
        if (PB == 4) acc = acc >> 8;
        acc += (v4i){cqck, cqck, cqck, cqck};
        store_scores<DQ>(a, out0, s0, slot, n, g, acc);
    }
}

} // namespace

template <int PB, int LPR, bool DQ, bool U> hipError_t launch_staged(const SddmmArgs &a, int waves, hipStream_t s)
{
    dim3 grid((unsigned)a.n_shares, (unsigned)a.batch);
    constexpr int STAGE = (LPR == 4) ? 4096 : (LPR == 64 ? 16384 : 8192);
    if (LPR == 64 && waves > 4) waves = 4;      // 64 KB of stages per workgroup
    if constexpr (!U) {
        if (a.kmat_rows <= (1 << 24) && a.ldk_bytes < (1 << 24) && (a.kmat_rows - 1) * a.ldk_bytes + a.row_bytes < ((int64_t)1 << 32)) {
            return launch_kernel((sddmm_staged_kernel<PB, LPR, DQ, U, true>), grid, dim3(64 * waves), waves * STAGE, s, a);
        }
    }
    return launch_kernel((sddmm_staged_kernel<PB, LPR, DQ, U, false>), grid, dim3(64 * waves), waves * STAGE, s, a);
}

template <int PB, bool DQ, bool U> hipError_t launch_sddmm_bits(const SddmmArgs &a, int waves, hipStream_t s)
{
    if (waves > 0) {
        if constexpr (PB == 4) {
            if (a.row_bytes == 32) { // 64 nibbles: one MFMA step
                dim3 grid((unsigned)a.n_shares, (unsigned)a.batch);
                switch (waves) {
                case 1: return launch_kernel((sddmm_nib32_kernel<1, DQ, U>), grid, dim3(64), 0, s, a);
                case 2: return launch_kernel((sddmm_nib32_kernel<2, DQ, U>), grid, dim3(128), 0, s, a);
                case 4: return launch_kernel((sddmm_nib32_kernel<4, DQ, U>), grid, dim3(256), 0, s, a);
                default: return launch_kernel((sddmm_nib32_kernel<8, DQ, U>), grid, dim3(512), 0, s, a);
                }
            }
        }
        // the narrowest stage that holds the row
        if (a.row_bytes <= 64 && PB != 16) return launch_staged<(PB == 16 ? 8 : PB), 4, DQ, U>(a, waves, s);
        if (a.row_bytes <= 128) return launch_staged<PB, 8, DQ, U>(a, waves, s);
        if (a.row_bytes <= 256) return launch_staged<PB, 16, DQ, U>(a, waves, s);
        if (a.row_bytes <= 512) return launch_staged<PB, 32, DQ, U>(a, waves, s);
        if (a.row_bytes <= 1024) return launch_staged<PB, 64, DQ, U>(a, waves, s);
    }
    dim3 grid((unsigned)a.n_shares, (unsigned)a.batch), block(64 * SDDMM_WAVES);
    if constexpr (U) {
        return launch_kernel((sddmm_unsigned_kernel<PB, DQ>), grid, block, 0, s, a); // any row length, operands straight from memory
    } else {
        const int kc = (a.row_bytes + StepBytes<PB>::value - 1) / StepBytes<PB>::value;
        if (kc == 1) return launch_kernel((sddmm_direct_kernel<PB, 1, DQ>), grid, block, 0, s, a);
        if (kc == 2) return launch_kernel((sddmm_direct_kernel<PB, 2, DQ>), grid, block, 0, s, a);
        if (kc <= 4) return launch_kernel((sddmm_direct_kernel<PB, 4, DQ>), grid, block, 0, s, a);
        return launch_kernel((sddmm_direct_kernel<PB, 0, DQ>), grid, block, 0, s, a);
    }
}

template <bool DQ> hipError_t launch_sddmm_out(int bits, const SddmmArgs &a, int waves, hipStream_t s)
{
    if (a.lhs_unsigned || a.rhs_unsigned) {
        if (bits == 8) return launch_sddmm_bits<8, DQ, true>(a, waves, s);
        if (bits == 4) return launch_sddmm_bits<4, DQ, true>(a, waves, s);
        return hipErrorInvalidValue;
    }
    if (bits == 4) return launch_sddmm_bits<4, DQ, false>(a, waves, s);
    if (bits == 16) return launch_sddmm_bits<16, DQ, false>(a, waves, s);
    return launch_sddmm_bits<8, DQ, false>(a, waves, s);
}

hipError_t launch_sddmm(int bits, const SddmmArgs &a, int waves, hipStream_t s)
{
    if (a.n_shares == 0 || a.batch == 0) return hipSuccess;
    return a.float_out ? launch_sddmm_out<true>(bits, a, waves, s) : launch_sddmm_out<false>(bits, a, waves, s);
}
