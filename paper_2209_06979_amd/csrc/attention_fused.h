// Fused quantized sparse self-attention for gfx950 (paper, Section 5.3): for one head and
// one row panel of the mask ONE WAVEFRONT runs SDDMM -> softmax -> int8 codes -> SpMM with
// the scores, probabilities and codes never leaving registers / LDS.  Latency is hidden by
// keeping a dozen such waves resident per CU, each with chunks of gathered rows in flight.
//
//   phase K  per chunk of 64 mask vectors: the Kmat rows named by the column indices are
//            copied from global memory straight into LDS (global_load_lds, no registers in
//            between); one v_mfma_i32_16x16x64_i8 per 16 vectors and 64 elements of the head
//            dimension gives the scores (head dim 64 = one MFMA, 128 = two; both operands are
//            contiguous along the reduction, Section 4.3).
//            The 8 Q rows sit in MFMA rows 0..7 for even tiles and in rows 8..15 for odd
//            tiles, so two tiles share one accumulator and all 64 lanes carry real scores.
//   softmax  fp32, base 2, over the panel's stored entries: in-lane over the tiles, DPP
//            rotations over the 16 lanes of a row, one cross-lane exchange for the two
//            tile parities; codes = clamp(rint(p / s_p), 0, 127) go to LDS as
//            [slot][8 rows] bytes (one 32-bit write per 4 codes).
//   phase V  SpMM (Section 4.2) per chunk: V rows are copied into the same LDS stages;
//            ds_read_b64_tr_b8 delivers both MFMA operands in place: the codes transposed
//            to [row][16 slots] and the V rows transposed to [column][16 slots].
//   output   the 8 x dk tile goes through LDS once to be stored as fp32 with 16-byte stores.
//
// Two variants (HPW = heads per workgroup):
//   HPW 1  any layout: the wave gathers the rows of its own head (64 bytes; 128 bytes for head
//          dimension 128 with 8-bit inputs) into its one LDS stage (5 KB of LDS per wave and
//          16 waves per CU for 64-byte rows).
//   HPW 2  token-major layout (the heads of a token are contiguous, as a QKV projection
//          writes them): two waves own two neighbouring heads and gather their 128 bytes of
//          a token with ONE request.  The L2 serves a 128-byte line at the cost of a 64-byte
//          half, so this halves the number of gather requests, which is what bounds the
//          kernel.  Each wave copies half of a chunk's rows; one s_barrier per chunk.
// LDS rows are as long as a gathered row (ROWB = HPW times the bytes of one head's row: 32 .. 128);
// slot s of a chunk lives in row (s % NIT) * (64/NIT) + s / NIT (NIT = ROWB/16 copy instructions
// per chunk, so that the column indices a lane needs are consecutive) and its 16-byte segments are
// XOR-swizzled with s % NIT so that rows read together fall into different banks.
#pragma once
#include "attention_order.h"
#include "internal.h"
#include "lds_async.h"
#include <type_traits>

namespace {

using namespace mcu;

// max / sum over the 16 lanes of a DPP row via rotations by 1, 2, 4, 8 (VALU only)
template <int CTRL> __device__ __forceinline__ float dpp_rot(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_max(float v)
{
    v = fmaxf(v, dpp_rot<0x121>(v)); // row_ror:1
    v = fmaxf(v, dpp_rot<0x122>(v));
    v = fmaxf(v, dpp_rot<0x124>(v));
    v = fmaxf(v, dpp_rot<0x128>(v));
    return v;
}
__device__ __forceinline__ int row16_imax(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, false)); // row_ror:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false));
    return v;
}
__device__ __forceinline__ float row16_sum(float v)
{
    v += dpp_rot<0x121>(v);
    v += dpp_rot<0x122>(v);
    v += dpp_rot<0x124>(v);
    v += dpp_rot<0x128>(v);
    return v;
}

// the values that lanes l and l + 32 hold, in both (in registers; through LDS the two exchanges of the softmax cost a round trip each)
__device__ __forceinline__ void both_halves(unsigned v, unsigned &lo, unsigned &hi)
{
    const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    lo = s[0];
    hi = s[1];
}

constexpr unsigned PAIR_ROWS_Y = 32768; // rows of the grid along y, the rest of them along z

// MAXCH: longest panel in chunks of 64 vectors.  HPW: heads (= waves) per workgroup.
// PB: bits of the re-quantised softmax output.  16 ("16b-8b" layer): the code c <= 32639 is split
// into signed bytes c = 256*hi + lo (Section 4.4); the lo codes of row r feed MFMA row 2r and the hi
// codes row 2r + 1 of the same instruction, and the output is (O_hi << 8) + O_lo.  The two sums of an output lie in neighbouring registers
// of a lane, a code's two bytes stay together from the rounded product to LDS, and the output tile has 8 rows.  (With a plane of
// its own for each, 8 rows apart: eight more byte permutations and stores of LDS a chunk, a tile of 16 rows to write, to add up between the waves and to
// put together; replayed from a graph 8 x 4 heads x 8192, (L, heads, dk) 169.3 -> 167.6 us, 1 x 368 x 112 4.37 -> 4.20, 1 x 1368 x 64 of nibbles
// 4.26 -> 4.06, 2 x 12 x 1016 x 80 14.4 -> 14.2.)
// QB: bits of Q, Kmat and V.  4 ("8b-4b" layer): rows are 32 bytes of packed nibbles, whose bytes are widened in registers (Section 4.4
// without an int4 matrix unit): the even elements of a 16-byte piece in lane groups 0 and 1, the odd ones in groups 2 and 3.  An
// odd element stays in the upper half of its byte, worth 16 x its value; an even one in the lower half as value + 8, which one
// three-input logic operation makes of it, where a shift to the upper half took two (and a select between the two kinds of lane a third).
// The scores come out 16-fold and the 8s as a constant per row of Q, with which the sums start; in the output the 8s are 8 times the sum of
// the codes, which one more MFMA per chunk adds up.  Short of the largest launches, which wait for L2 (a request per row whatever its
// length), these layers are bound by the VALU: a chunk took 64 + 32 + 45 instructions, now 24 + 32 + 37.  By itself, 8-bit codes:
// 8 heads x 1752, dk = 128, 73 % empty 14.3 -> 12.0 us; 12 x 4064, dk = 128, 80 % 60.4 -> 54.3; 8 x 12 x 1712, dk = 96, 72 % 110.6 -> 99.6;
// 8 x 12 x 5432, dk = 64, 92 % 199 both.
// KS: waves that share one (panel, head) when a panel is longer than MAXCH chunks: wave ks takes
// chunks ks, ks + KS, ...; the waves exchange their row maxima and row sums through LDS and add up
// their partial output tiles at the end (three workgroup barriers in total).  With HPW 2 the
// workgroup has 2 * KS waves: pair ks (one wave per head) gathers its chunks into its own two
// stages, and since the per-chunk barrier is the workgroup's, every wave goes through the chunk
// loops as often as the pair with the most chunks does.
// DK: head dimension, 64 or 128; 192: always PAD, dimensions of 144 to 192 in LDS rows of 256 bytes (128 for nibbles) and two waves
// per SIMD, 1.2 - 2.3 times faster than separate kernels (8 heads x 4096, dk = 160: 87 -> 50 us).  Rows of 128 bytes (DK 128, 8-bit inputs) are gathered by one head per
// workgroup only; the 64-byte rows of DK 128 with 4-bit inputs behave like those of DK 64 with 8-bit ones.
// PAD: the head dimension is smaller than DK (any multiple of 16, of 32 for 4-bit inputs): a row has only
// a.real_pieces 16-byte pieces.  The copies of the missing pieces are left out, so the places they would
// land in keep the zeros written once at the start (place p of an LDS row always receives the same piece
// number, see the copy layout below); the Q registers of those pieces are zero as well.  Zero columns add
// nothing to a score and give zero output columns, which are not stored.  Two heads per workgroup (DK 64 only): the places of both heads' pieces,
// which are contiguous in memory, side by side as if the rows were full.
template <int MAXCH, int HPW, int PB, int QB, int KS, int DK, bool PAD = false>
__global__ __launch_bounds__(64 * HPW * KS, (((HPW == 1 && PB == 8 && KS == 1 && DK == 64) || (HPW == 2 && DK == 64)) ? 4 : ((KS == 8 || DK == 192) ? 2 : 3)))
void attention_fused_kernel(AttnArgs a)
{
    static_assert(!PAD || HPW == 1 || DK == 64, "shorter rows of more than 64 elements: one head per workgroup");
    static_assert(PB == 8 || PB == 16, "8- or 16-bit codes");
    static_assert(QB == 8 || QB == 4, "Q, K, V are 8-bit or packed 4-bit");
    static_assert(DK == 64 || (DK == 128 && (QB == 4 || HPW == 1)) || (DK == 192 && PAD), "rows of 128 bytes: one head per workgroup");
    constexpr int NW = HPW * KS;         // waves per workgroup
    constexpr int OTILE = 8 * (DK + 4) * 4;                                         // a wave's output tile, staged where the gathered rows were
    // The code area holds ONE chunk, [slot][8 rows][1 or 2 bytes] (codes are written right before they are read; an area for all chunks and
    // the output tile took 3.5 - 14 KB more of LDS per wave): a workgroup of two heads stays below 20 KB, eight of them, i.e. all 2048 of a 8 x 4096
    // layer, are resident at once; four waves of a dk of 144 - 192 take 68 KB instead of 82, two workgroups a compute unit instead of
    // one (12 heads x 5568, dk = 144, 77 % empty 489 -> 296 us, 3 x 2264, dk = 160 28.5 -> 19.1); with 16-bit codes 16 waves are resident instead of
    // 13 (8 heads x 5008, dk = 96, 95 % 29.1 -> 25.3; 12 x 2 x 2336, dk = 64, 4-bit inputs 35.8 -> 33.7).
    constexpr int SLOTB = PB, PLB = 64 * SLOTB;                                     // bytes of a slot's codes; of that area
    constexpr int DKB = DK * QB / 8; // bytes of one head's row
    constexpr int KK = DK / 64;      // MFMA steps along the head dimension
    constexpr int NO = DK / 16;      // column tiles of the output
    constexpr int NPR = MAXCH * 2;   // pairs of score tiles
    constexpr int ROWB = DK == 192 ? 32 * QB : DKB * HPW;  // bytes of a gathered row's place in LDS: a power of two
    constexpr int LPR = ROWB / 16;   // lanes per row
    constexpr int NIT = LPR;         // copy instructions per chunk
    constexpr int NITW = NIT / HPW;  // ... of which each wave issues this many (4; 2 for nibbles; 8 for head dimension 128)
    constexpr int NCT = QB == 8 ? NO : NO / 2; // 16-byte pieces of a row that become output columns
    constexpr int SWZ = LPR - 1;
    constexpr int NIB = (int)0xF0F0F0F0;
    constexpr int STG = 64 * ROWB;   // bytes of one stage
    constexpr int NST = HPW;         // stages: one for a lone wave, two when two waves share the chunks
    constexpr int WSTG = (HPW == 1 && OTILE > STG) ? OTILE : NST * STG;               // ... of the stages of one share of the chunks
    static_assert(HPW == 1 || OTILE <= STG, "with two heads per workgroup a wave's output tile is staged in one gather stage");
    __shared__ __attribute__((aligned(16))) char stage_all[WSTG * KS];       // chunks of gathered rows (KS > 1: one stage per wave)
    __shared__ __attribute__((aligned(16))) char Pl_all[NW * PLB]; // codes of a chunk, per wave
    __shared__ __attribute__((aligned(8))) char zeros[72];                     // row operand of the MFMA rows that carry no codes
    __shared__ int xch[2][HPW][KS][8];                                        // row maxima / row sums of the KS waves of a head

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = (HPW > 1) ? wave % HPW : 0;  // head within the workgroup
    const int ks = (KS > 1) ? wave / HPW : 0;  // share of the panel's chunks
    char *stage = stage_all + ks * WSTG;
    const int j = lane & 15, g = lane >> 4;
    const int rg = lane / LPR, seg = lane % LPR;
    // Workgroups are handed to the 8 XCDs round-robin by linear id.  1, 2, 4 or 8 (head group, batch item) pairs are worked on
    // at a time, a row of the grid (attention_pair_shift): an XCD then sees one pair at a time, and neighbouring ones one after the other.
    // In (L, heads, dk) tensors neighbouring heads share lines unless their rows are whole ones: an XCD finds in its L2 what it would
    // otherwise fetch while another XCD fetches it, too.  (By itself, neighbouring pairs at the same time and as it is: 8 x 8 heads x 1800, 87 %
    // empty, 8-bit codes and inputs, dk = 32 36.6 -> 33.9 us, 48 60.2 -> 41.6, 80 61.8 -> 55.4, 96 63.1 -> 59.0, 128 52.4 -> 50.3.)
    const int groups = a.heads / HPW;
    // (all that a wave needs first in one round trip, not one by one as it comes to be needed: the first line of arguments and what follows it, which no
    // argument that only some kernels read may part.  With the panels' length among the pointers behind that line the kernels that do not read it waited
    // a second and a third time; 4 heads x 1000 4.31 -> 4.18 us, 2 heads x 520 3.65 -> 3.53, 8 x 4 heads x 8192 of any kind 0.994 - 1.002x.)
    constexpr bool COMPUTED = !(HPW == 2 && KS > 1 && PB == 8 && QB == 8 && !PAD); // (see below)
    if constexpr (COMPUTED) asm volatile("" ::"s"(a.uniform_vectors));
    asm volatile("" ::"s"(a.panel_ptr), "s"(a.slot_idx), "s"(a.panel_list), "s"(a.heads), "s"(a.batch), "s"(a.pair_shift), "s"(a.pair_rows),
                 "s"(a.Km), "s"(a.in_token_stride), "s"(a.in_head_stride), "s"(a.Q));
    const int grid_row = (int)(blockIdx.z * PAIR_ROWS_Y + blockIdx.y);
    if (grid_row >= a.pair_rows) return;
    const int pair = (int)(blockIdx.x & ((1u << a.pair_shift) - 1)) * a.pair_rows + grid_row;
    int hgrp = pair, item = 0;
    if (a.batch > 1) {
        item = pair / groups;
        hgrp = pair - item * groups;
    }
    const int panel = a.panel_list ? a.panel_list[blockIdx.x >> a.pair_shift] : (int)(blockIdx.x >> a.pair_shift);
    const int head = hgrp * HPW + w;
    // (panels of equal length: first slot and length without a trip to memory that the column indices wait for.  Replayed from a graph, three layers
    // in turn: 4 heads x 1000 4.46 -> 4.40 us, 8 x 4 heads x 8192, 16-bit codes, (L, heads, dk) 170.5 -> 169.3; as single calls the same, the host issues them.
    // Not where several waves share the 8-bit codes of a pair: all 128 registers are taken there, and one more would be spilled.)
    int s0, n = COMPUTED ? a.uniform_vectors : 0;
    if (COMPUTED && n > 0) s0 = panel * ((n + MC_CHUNK - 1) / MC_CHUNK * MC_CHUNK);
    else {
        s0 = a.panel_ptr[2 * panel];
        n = a.panel_ptr[2 * panel + 1] - s0;
    }
    const int nch = (n + MC_CHUNK - 1) / MC_CHUNK;
    const int32_t *idx = a.slot_idx + s0;
    const int64_t goff = (int64_t)hgrp * HPW * a.in_head_stride; // first head of the group
    const int64_t boff = (int64_t)item * a.in_batch_stride; // batch item
    const uint8_t *Kg = a.Km + boff + goff, *Vg = a.Vm + boff + goff;
    float *Oh = a.O + (int64_t)item * a.batch_stride + (int64_t)head * a.head_stride + (int64_t)panel * 8 * a.token_stride;
    char *Pl = Pl_all + wave * PLB;
    const int nloc = (nch > ks) ? (nch - ks + KS - 1) / KS : 0; // chunks of this wave: ks, ks + KS, ...
    // Waves that meet at a workgroup barrier per chunk all make as many passes as the busiest of them
    // (a pass without a chunk of its own is the barrier alone).
    constexpr bool LOCKSTEP = (HPW > 1 && KS > 1);
    const int npass = LOCKSTEP ? (nch + KS - 1) / KS : nloc;
    if (PB == 8 && lane < 18) reinterpret_cast<int *>(zeros)[lane] = 0; // every wave writes the same zeros: no race that matters
    if (PAD) {
        // the places of the pieces a row does not have: zero once, never written again
        for (int i = threadIdx.x; i < WSTG * KS / 16; i += 64 * NW) reinterpret_cast<v4i *>(stage_all)[i] = (v4i){0, 0, 0, 0};
        __syncthreads(); // (waits for the writes, too: the copies below must land after them)
    }

    // Q rows twice: in MFMA rows 0..7 (q_lo) and in rows 8..15 (q_hi)
    v4i q_lo[KK], q_hi[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        const uint8_t *qrow = a.Q + boff + (int64_t)head * a.in_head_stride + (int64_t)(panel * 8 + (j & 7)) * a.in_token_stride;
        v4i qv = {0, 0, 0, 0};
        if (!PAD || (QB == 8 ? 4 * kk + g : 2 * kk + (g & 1)) < a.real_pieces) { // (a piece the row does not have stays zero)
            if (QB == 8) {
                qv = *reinterpret_cast<const v4i *>(qrow + kk * 64 + g * 16);
            } else { // 16 x the even elements; the odd ones as they are, sign-extended from the upper half
                const v4i raw = *reinterpret_cast<const v4i *>(qrow + kk * 32 + (g & 1) * 16);
                qv = (g < 2) ? ((raw << 4) & NIB) : ((((((raw >> 4) & ~NIB) ^ 0x08080808) | (int)0x80808080) - 0x08080808) ^ (int)0x80808080);
            }
        }
        q_lo[kk] = (j < 8) ? qv : (v4i){0, 0, 0, 0};
        q_hi[kk] = (j < 8) ? (v4i){0, 0, 0, 0} : qv;
    }
    // Copy instruction i of a chunk: lane (rg, seg) fetches segment seg ^ i of the row in slot
    // rg*NIT + i; it lands in LDS row i*(64/NIT) + rg.  Wave w issues instructions NITW*w .. +NITW-1,
    // whose column indices are consecutive slots: one 128-bit (64-bit) index load per chunk.
    constexpr int SHARE = NITW >= 4 ? 4 : 2, NIX = NITW / SHARE;  // lanes that share their indices; indices a lane loads per chunk
    static_assert(SHARE <= LPR, "only lanes of one row share");
    typedef int ixv_t __attribute__((ext_vector_type(NIX)));
    unsigned segoff[NITW];
#pragma unroll
    for (int i = 0; i < NITW; ++i) {
        const int place = seg ^ ((NITW * w + i) & SWZ);
        segoff[i] = place * 16;
        if (PAD) { // a piece that the row does not have is not fetched (the sign says so)
            const int piece = HPW == 1 ? place : place % NITW;
            segoff[i] = (HPW == 1 ? place : place / NITW * a.real_pieces + piece) * 16;
            if (piece >= a.real_pieces) segoff[i] |= 1u << 31;
        }
    }
    const unsigned stage_u = lds_addr_uniform(stage);  // this wave's stage(s)
    // A lane's copies take NITW indices, the same for all lanes of a row.  Loaded by each lane they would be a fifth of
    // all bytes that L1 returns: a lane loads NIX of them and takes the others from its neighbours.  (By itself: 8 x 4 heads x 8192,
    // (L, heads, dk), 181 -> 177 us; 8 heads x 4096 x 128 22.6 -> 22.1; (heads, L, dk) tensors of dk = 64 0 - 1 %.)
    // (a chunk's place is wave-uniform: a scalar base and the lane's constant offset)
    const unsigned lane_idx = (rg * NIT + NITW * w + (lane % SHARE) * NIX) * 4;
    auto index_of = [&](auto I, const ixv_t &ix) -> unsigned { // index of copy instruction i
        constexpr int i = decltype(I)::value, q = i / NIX, ctrl = SHARE == 4 ? q * 0x55 : (q == 0 ? 0xA0 : 0xF5); // quad_perm [q,q,q,q] / [0,0,2,2], [1,1,3,3]
        return (unsigned)__builtin_amdgcn_mov_dpp(ix[i % NIX], ctrl, 0xF, 0xF, true);
    };
    auto load_idx = [&](int c) -> ixv_t {
        return *reinterpret_cast<const ixv_t *>(reinterpret_cast<const char *>(idx + c * MC_CHUNK) + lane_idx);
    };
    const unsigned tstride = (unsigned)a.in_token_stride;
    // issue(c, st): this wave's copies of chunk c into stage st, from the column indices held
    // in ixn; then the indices of the following chunk are requested (an ordinary load that has
    // long arrived by the time they are needed: a vm_wait<0>() lies in between).
    ixv_t ixn = {};
    auto issue = [&](const uint8_t *base, int c, int st) {
        ixv_t row;                             // (multiplied by the lane that holds an index, handed over in the sum)
#pragma unroll
        for (int q = 0; q < NIX; ++q) row[q] = (int)__umul24((unsigned)ixn[q], tstride);
        static_for<NITW>([&](auto I) {
            constexpr int i = decltype(I)::value;
            unsigned off = segoff[i];
            if (PAD) asm("" : "+v"(off)); // (sixteen conditions kept would be more than the scalar registers)
            const unsigned at = index_of(I, row) + off; // (the exchange with all lanes active)
            if (!PAD || (int)off >= 0) copy16_to_lds(base, at, stage_u + st * STG + (NITW * w + i) * 1024);
        });
        ixn = load_idx((c + KS < nch) ? c + KS : c);
    };
    ixv_t ix_first = {};                           // the first chunk's indices, for K and V
    if (nloc > 0) ix_first = load_idx(ks);
    auto start_pipeline = [&](const uint8_t *base) {
        lgkm_wait();                               // no read of the stage is still in flight
        if (HPW > 1) __builtin_amdgcn_s_barrier(); // both waves are done with the stages
        if (nloc > 0) {
            ixn = ix_first;
            issue(base, ks, 0);
        }
    };
    // Makes chunk c readable.  HPW 1: the next chunk is issued by release() once this one has
    // been read.  HPW 2: both halves have landed after the barrier, which also tells that
    // everybody is done reading the pair's previous chunk, so its next chunk can go into the other
    // stage st now.  (c may lie beyond the panel's last chunk in a pass of waiting only.)
    auto acquire = [&](const uint8_t *base, int c, int st) {
        vm_wait<0>();
        if (HPW > 1) {
            __builtin_amdgcn_s_barrier();
            if (c + KS < nch) issue(base, c + KS, st);
        }
    };
    auto release = [&](const uint8_t *base, int c) { // the reads of chunk c have been issued
        if (HPW == 1 && c + KS < nch) {
            lgkm_wait(); // ... and have returned: the one stage may be overwritten
            issue(base, c + KS, 0);
        }
    };

    // ---- phase K: scores; lane (j, g) owns row 4*(g&1) + r of tile 2*pr + (g >> 1) -----
    // The integer scores stay in registers; only the last chunk can hold padded slots, which
    // are kept out of the row sum (and so out of the codes) below.
    // K operand of tile tl: slot s = tl*16 + j sits in LDS row (s % NIT)*(64/NIT) + s/NIT,
    // i.e. byte (j % NIT)*1024 + (j / NIT)*ROWB + tl*256; segment (NITW*w + piece) ^ (j % NIT), where
    // lane group g reads piece 4*kk + g of its head's row in MFMA step kk (8 bit) or piece 2*kk + g % 2
    // (4 bit: even elements of the piece for g < 2, odd elements for g >= 2, as on the Q side)
    const char *kaddr[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        kaddr[kk] = stage + (j % NIT) * 1024 + (j / NIT) * ROWB + (((NITW * w + (QB == 8 ? 4 * kk + g : 2 * kk + (g & 1))) ^ (j % NIT)) * 16);
    const int flip = g < 2 ? 0x08080808 : 0, half = g < 2 ? ~NIB : NIB;
    auto kop = [&](v4i raw) -> v4i {
        if (QB == 8) return raw;
        return (raw ^ flip) & half;
    };
    // What the sums start with: the bit pattern of 1.5 * 2^23 -- as a float a sum then is that much more than its value, exactly, and no conversion
    // is needed -- and, 4 bit, -8 x 16 x the row's even elements.  (Scores stay below 2^22: 192 x 128 x 128.)
    static_assert(DK * 128 * 128 < 1 << 22, "scores are exact beside 1.5 * 2^23");
    // (A conversion takes a SIMD 4.3 clocks, as a byte permutation, a multiply-add of integers or an exchange of neighbours; a sum or product of floats 2.3 -
    // 2.7, an exponential 8.9.  With one product per index instead of per copy and codes by one multiply-add and permutations, 40
    // layers replayed from graphs 1.010x in the mean, 8 x 4 heads x 8192 with 16-bit codes 1.02, 0.99 - 1.05x: it is the gather that takes the time.)
    // FOLDED: subtraction and product of the softmax in one multiply-add (below): the pairs by several waves with 16-bit codes, which the instructions
    // bound, too (three operations a score with conversions 169.7 us at 8 x 4 heads x 8192, subtraction and product 172, folded 168.2).  Elsewhere the exact
    // difference gives the largest term of a row exactly, at up to 0.5 % of the time.
    constexpr bool FOLDED = HPW == 2 && KS > 1 && PB == 16 && QB == 8;
    constexpr int FLOAT0 = 0x4B400000;
    v4i first = {FLOAT0, FLOAT0, FLOAT0, FLOAT0};
    if (QB == 4) {
        const int minus8 = g < 2 ? (int)0xF8F8F8F8 : 0;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            first = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_lo[kk], (v4i){minus8, minus8, minus8, minus8}, first, 0, 0, 0);
            first = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_hi[kk], (v4i){minus8, minus8, minus8, minus8}, first, 0, 0, 0);
        }
    }
    v4i sc[NPR];
    int imax[4] = {INT32_MIN, INT32_MIN, INT32_MIN, INT32_MIN};
    const int tail = n - (nch - 1) * MC_CHUNK; // real vectors in the last chunk
    bool keep[2];                               // this lane's slots of the last chunk are real
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) keep[pr] = (2 * pr + (g >> 1)) * 16 + j < tail;
    start_pipeline(Kg);
    // (from here on c counts this wave's chunks; gc is the chunk's number in the panel)
    static_for<MAXCH>([&](auto C) {
        constexpr int c = C, ST = (c % NST) * STG;
        const int gc = ks + c * KS;
        if (c < npass) {
            acquire(Kg, gc, (c + 1) % NST);
            if (LOCKSTEP && c >= nloc) return;
            v4i kt[KK][4]; // tiles 0..3 of the chunk
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int tl = 0; tl < 4; ++tl) kt[kk][tl] = *reinterpret_cast<const v4i *>(kaddr[kk] + ST + tl * 256);
            release(Kg, gc);
            sc[2 * c] = first;
            sc[2 * c + 1] = first;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                sc[2 * c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_lo[kk], kop(kt[kk][0]), sc[2 * c], 0, 0, 0);
                sc[2 * c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_hi[kk], kop(kt[kk][1]), sc[2 * c], 0, 0, 0);
                sc[2 * c + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_lo[kk], kop(kt[kk][2]), sc[2 * c + 1], 0, 0, 0);
                sc[2 * c + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q_hi[kk], kop(kt[kk][3]), sc[2 * c + 1], 0, 0, 0);
            }
            // a padded slot repeats the panel's last real column, so its score duplicates a real
            // one and cannot change the row maximum: no masking here
#pragma unroll
            for (int r = 0; r < 4; ++r) imax[r] = max(imax[r], max(sc[2 * c][r], sc[2 * c + 1][r]));
        }
    });
    // all Kmat rows are consumed: start copying V rows while the softmax runs
    start_pipeline(Vg);

    // ---- softmax over row 4*(g&1) + r, in base 2: exp(x - max) = 2^((s - smax) * scale2), the difference exact -----
    // (FOLDED: s * scale2 - m2 by one multiply-add, exact but for its rounding and for what m2 = smax * scale2, both with their 1.5 * 2^23, was rounded
    // by.  That is the same for the whole row, a factor of 2^32 at most, which the sum takes off again, because a scale of 64 leaves the largest scores
    // alone as any larger one does: what is one less is 2^-64 of them, which no sum of 4096 holds, and no code shows it while inv_s_p is at most
    // FOLDED_MAX_INV_S_P, nor what the factor of 2^-32 takes from entries below 2^-94: larger ones are not launched here.  Error against 64 bits, six layers of 2000 - 3400
    // tokens: 2.86e-5, 2.89e-5 with conversions.)
    constexpr float LOG2E = 1.4426950408889634f;
    const float scale2 = fminf(a.score_scale * LOG2E * (QB == 4 ? 0.0625f : 1.f), FOLDED ? 64.f : 256.f);
    float top[4], srow[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        unsigned lo, hi;
        both_halves((unsigned)row16_imax(imax[r]), lo, hi);
        imax[r] = max((int)lo, (int)hi);
    }
    if (KS > 1) { // row 4*(g&1) + r: lanes 0 and 16 publish, everybody reads all waves
        if (lane == 0 || lane == 16) {
#pragma unroll
            for (int r = 0; r < 4; ++r) xch[0][w][ks][4 * (g & 1) + r] = imax[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < KS; ++k) imax[r] = max(imax[r], xch[0][w][k][4 * (g & 1) + r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) top[r] = FOLDED ? __builtin_bit_cast(float, imax[r]) * scale2 : __builtin_bit_cast(float, imax[r]);
    float x[NPR][4];
    static_for<MAXCH>([&](auto C) {
        constexpr int c = C;
        if (c < nloc) {
#pragma unroll
            for (int pr = 0; pr < 2; ++pr)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int sum = sc[2 * c + pr][r]; // (a bit cast of a vector's element takes the first one)
                    x[2 * c + pr][r] = __builtin_amdgcn_exp2f(FOLDED ? __builtin_fmaf(__builtin_bit_cast(float, sum), scale2, -top[r]) : (__builtin_bit_cast(float, sum) - top[r]) * scale2);
                }
            if (ks + c * KS == nch - 1) {
                // the panel's last chunk: padded slots count for nothing.  (The empty statement keeps
                // this a branch taken once per wave instead of selects in every chunk.)
                asm volatile("" ::: "memory");
#pragma unroll
                for (int pr = 0; pr < 2; ++pr)
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[2 * c + pr][r] = keep[pr] ? x[2 * c + pr][r] : 0.f;
            }
#pragma unroll
            for (int pr = 0; pr < 2; ++pr)
#pragma unroll
                for (int r = 0; r < 4; ++r) srow[r] += x[2 * c + pr][r];
        }
    });
    float rinv[4]; // p / s_p = e * (1 / (sum * s_p)): one division per row instead of one per entry
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        unsigned lo, hi;
        both_halves(__builtin_bit_cast(unsigned, row16_sum(srow[r])), lo, hi);
        srow[r] = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
    }
    if (KS > 1) { // every wave adds the partial sums in the same order: identical totals everywhere
        if (lane == 0 || lane == 16) {
#pragma unroll
            for (int r = 0; r < 4; ++r) xch[1][w][ks][4 * (g & 1) + r] = __builtin_bit_cast(int, srow[r]);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            srow[r] = 0.f;
#pragma unroll
            for (int k = 0; k < KS; ++k) srow[r] += __builtin_bit_cast(float, xch[1][w][k][4 * (g & 1) + r]);
        }
    }
    {   // one division per lane, of the row that its place in a group of four names
        const float s01 = (lane & 1) ? srow[1] : srow[0], s23 = (lane & 1) ? srow[3] : srow[2];
        const int q = __builtin_bit_cast(int, a.inv_s_p / ((lane & 2) ? s23 : s01));
        rinv[0] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, q, 0x00, 0xF, 0xF, false)); // quad_perm [0,0,0,0]
        rinv[1] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, q, 0x55, 0xF, 0xF, false));
        rinv[2] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, q, 0xAA, 0xF, 0xF, false));
        rinv[3] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, q, 0xFF, 0xF, 0xF, false));
    }
    // ---- phase V: O = codes * V ------------------------------------------------------------------
    v4i o[NO];
#pragma unroll
    for (int ct = 0; ct < NO; ++ct) o[ct] = (v4i){0, 0, 0, 0};
    v4i ocodes = {0, 0, 0, 0};                 // 4 bit: sums of the codes
    // Lane (g, src) supplies the V rows of the chunk's slots s = g*16 + ii and s + 8, and their codes.  (8 slots on is
    // 8 / NIT rows of the stage on, 64 bytes of codes on: instruction offsets; the swizzled places of the column tiles
    // are worked out once.)
    const int src = lane & 15, ii = src >> 1, slot0 = g * 16 + ii;
    // (rows of 256 bytes: 8 slots on is 8 copy instructions on, whose swizzle differs in its top bit.)
    constexpr int ROWS8 = NIT == 16 ? 8 * 1024 : 8 / NIT * ROWB;
    const char *vaddr[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
        vaddr[ct] = stage + (slot0 % NIT) * 1024 + (slot0 / NIT) * ROWB + (((NITW * w + ct) ^ (slot0 % NIT)) * 16) + 8 * (src & 1);
    // lanes 2t and 2t+1 supply the 8-byte pieces that end up in MFMA rows 0..7 and 8..15: the
    // codes and 8 zero bytes (PB 8; they do not move from chunk to chunk), or the low and high bytes of rows 0..3 and 4..7 (PB 16)
    const char *paddr = (PB == 8 && (src & 1)) ? zeros : Pl + slot0 * SLOTB + (PB == 8 ? 0 : (src & 1) * 8);
    char *const code_at = Pl + ((g >> 1) * 16 + j) * SLOTB + SLOTB / 2 * (g & 1); // codes of tile pair pr: 32 slots * pr on
    // p / s_p stays within the largest code unless s_p is below its reciprocal
    const bool cap = a.inv_s_p > (PB == 8 ? 127.f : 32639.f);
    static_for<MAXCH>([&](auto C) {
        constexpr int c = C;
        const int gc = ks + c * KS;
        if (LOCKSTEP && c >= nloc) { // a pass of waiting only
            if (c < npass) acquire(Vg, gc, (c + 1) % NST);
            return;
        }
        if (c < nloc) {
            // Codes of this chunk's slots (tile*16 + j), rows 4*(g&1) .. +3: one 32-bit LDS write
            // (PB 16: one of 64 bits) per tile.  Done here, chunk by chunk, so that this ALU work overlaps the V copies in flight.
            auto make_codes = [&](auto Cap) {
                constexpr bool CAP = decltype(Cap)::value;
#pragma unroll
                for (int pr = 0; pr < 2; ++pr) {
                    // code = rint(x * rinv), ties to even: added to 1.5 * 2^23 the product becomes an integer in the low half of the word.
                    // 16 bit, plus 128: code = 256 * hi + lo with hi = (code + 128) >> 8 in [0, 127] then is the second byte and lo, in [-128, 127],
                    // the first one with its top bit flipped.
                    constexpr float INTEGER = PB == 8 ? 12582912.f : 12582912.f + 128.f;
                    unsigned u[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float e = x[2 * c + pr][r];
                        u[r] = __builtin_bit_cast(unsigned, CAP ? fminf(e * rinv[r], PB == 8 ? 127.f : 32639.f) + INTEGER : __builtin_fmaf(e, rinv[r], INTEGER));
                    }
                    char *to = code_at + pr * 32 * SLOTB;
                    if (PB == 8) {
                        const unsigned c01 = __builtin_amdgcn_perm(u[1], u[0], 0x05010400), c23 = __builtin_amdgcn_perm(u[3], u[2], 0x05010400);
                        *reinterpret_cast<unsigned *>(to) = __builtin_amdgcn_perm(c23, c01, 0x05040100);
                    } else {
                        *reinterpret_cast<v2i *>(to) = (v2i){(int)(__builtin_amdgcn_perm(u[1], u[0], 0x05040100) ^ 0x00800080u),
                                                             (int)(__builtin_amdgcn_perm(u[3], u[2], 0x05040100) ^ 0x00800080u)};
                    }
                }
            };
            if (cap) make_codes(std::true_type{});
            else make_codes(std::false_type{});
            acquire(Vg, gc, (c + 1) % NST);
            // the codes, transposed to the MFMA row operand: row j < 8, slots g*16 .. +15
            const v2i p0 = lds_read_tr8(paddr), p1 = lds_read_tr8(paddr + (PB == 8 ? 64 : 128));
            v2i d[NCT][2];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                d[ct][0] = lds_read_tr8(vaddr[ct] + (c % NST) * STG);
                if (NIT == 16) d[ct][1] = lds_read_tr8(stage + ((int)(vaddr[ct] - stage) ^ 128) + ROWS8);
                else d[ct][1] = lds_read_tr8(vaddr[ct] + (c % NST) * STG + ROWS8);
            }
            release(Vg, gc);
            if (HPW == 1) asm volatile("" ::: "memory"); // (the next chunk's codes go where this one's were read)
            const v4i aop = {p0.x, p0.y, p1.x, p1.y};
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const v4i bop = {d[ct][0].x, d[ct][0].y, d[ct][1].x, d[ct][1].y};
                if (QB == 8) {
                    o[ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop, bop, o[ct], 0, 0, 0);
                } else { // byte j of the piece holds columns 32*ct + 2j (low nibble) and 2j + 1 (high nibble)
                    o[2 * ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop, (bop ^ 0x08080808) & ~NIB, o[2 * ct], 0, 0, 0);
                    o[2 * ct + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop, bop & NIB, o[2 * ct + 1], 0, 0, 0);
                }
            }
            if (QB == 4) ocodes = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop, (v4i){0x01010101, 0x01010101, 0x01010101, 0x01010101}, ocodes, 0, 0, 0);
        }
    });

    // ---- output: 8 x DK tile through this wave's stage, scaled, 16-byte stores -------------
    vm_wait<0>();
    lgkm_wait();
    if (HPW == 2) {
        __builtin_amdgcn_s_barrier(); // nobody reads the stages any more: each wave takes one for its tile
    }
    int *Ol = reinterpret_cast<int *>(stage_all + ks * WSTG + w * STG); // (HPW 2: as many stages as waves)
    // lane (j, g) has rows 4g .. 4g+3, or (PB 16) the low and the high plane's sums of rows 2g and 2g + 1
    if (g < 2 || PB == 16) {
        constexpr int ROWS = PB == 8 ? 4 : 2;
#pragma unroll
        for (int ct = 0; ct < NO; ++ct) {
            // nibbles: low ones were 8 too large, high ones carry a factor 16; each plane's sum for itself
            auto sum = [&](int r) -> int { return QB == 8 ? o[ct][r] : (ct & 1) ? o[ct][r] >> 4 : o[ct][r] - 8 * ocodes[r]; };
            const int col = QB == 8 ? ct * 16 + j : (ct >> 1) * 32 + 2 * j + (ct & 1);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) Ol[(ROWS * g + r) * (DK + 4) + col] = PB == 8 ? sum(r) : (sum(2 * r + 1) << 8) + sum(2 * r);
        }
    }
    lgkm_wait();
    if (KS > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier();
    // the tile of wave k of this wave's head, and this thread's number among the 64 * KS threads of the head
    auto partial_tile = [&](int k) -> const int * {
        return reinterpret_cast<const int *>(stage_all + k * WSTG + w * STG);
    };
    const int tih = ks * 64 + lane;
    if (a.out_f16) {
        // fp16: 8 rows x DK/8 pieces of 8 columns, one 16-byte store each
#pragma unroll
        for (int h = 0; h < (DK + 64 * KS - 1) / (64 * KS); ++h) {
            const int piece = tih + h * 64 * KS;
            if (piece >= DK) continue;
            const int row = piece / (DK / 8), col = (piece % (DK / 8)) * 8;
            if (PAD && col >= a.out_cols) continue;
            v4h hv[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                v4i sres = {0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const int *Ok = (KS > 1) ? partial_tile(k) : Ol;
                    sres += *reinterpret_cast<const v4i *>(&Ok[row * (DK + 4) + col + 4 * q]);
                }
                hv[q] = to_half4((v4f){sres.x * a.out_scale, sres.y * a.out_scale, sres.z * a.out_scale, sres.w * a.out_scale});
            }
            typedef _Float16 v8h __attribute__((ext_vector_type(8)));
            const int64_t off = (Oh - a.O) + (int64_t)row * a.token_stride + col;
            __builtin_nontemporal_store((v8h){hv[0].x, hv[0].y, hv[0].z, hv[0].w, hv[1].x, hv[1].y, hv[1].z, hv[1].w},
                                        reinterpret_cast<v8h *>(reinterpret_cast<_Float16 *>(a.O) + off));
        }
        return;
    }
    // 8 rows x DK/4 pieces of 4 columns; with KS waves all threads share the adding up of the partial tiles
#pragma unroll
    for (int h = 0; h < (2 * DK + 64 * KS - 1) / (64 * KS); ++h) {
        const int piece = tih + h * 64 * KS;
        if (piece >= 2 * DK) continue;
        const int row = piece / (DK / 4), col = (piece % (DK / 4)) * 4;
        if (PAD && col >= a.out_cols) continue;
        v4i sres = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int *Ok = (KS > 1) ? partial_tile(k) : Ol;
            sres += *reinterpret_cast<const v4i *>(&Ok[row * (DK + 4) + col]);
        }
        const v4f f = {sres.x * a.out_scale, sres.y * a.out_scale, sres.z * a.out_scale, sres.w * a.out_scale};
        __builtin_nontemporal_store(f, reinterpret_cast<v4f *>(Oh + (int64_t)row * a.token_stride + col));
    }
}

template <int HPW, int PB, int QB, int KS, int DK, bool PAD> hipError_t launch_pairs(AttnArgs a, hipStream_t s)
{
    if (HPW == 2 && KS > 1 && PB == 16 && QB == 8 && !(a.inv_s_p <= FOLDED_MAX_INV_S_P)) return hipErrorInvalidValue;
    const unsigned pairs = (unsigned)(a.heads / HPW) * (unsigned)a.batch;
    a.pair_shift = attention_pair_shift(a, HPW, PAD ? a.real_pieces * 16 : DK * QB / 8);
    a.pair_rows = (int)(pairs >> a.pair_shift);
    const unsigned rows = (unsigned)a.pair_rows, y = rows < PAIR_ROWS_Y ? rows : PAIR_ROWS_Y;
    return launch_kernel((attention_fused_kernel<8, HPW, PB, QB, KS, DK, PAD>), dim3((unsigned)a.P << a.pair_shift, y, (rows + y - 1) / y),
                       dim3(64 * HPW * KS), 0, s, a);
}

} // namespace
