// SpMM with the dense operand resident in LDS, for matrices whose column indices name the rows of B many times over.
//
// The paper's kernel (Section 4.2) fetches, for every row panel, the B rows its vectors name and
// accepts that those rows have no reuse in on-chip memory.  On gfx950 a workgroup can hold
// 160 KB of LDS, and the transposing LDS read takes a per-lane address, so the "gather" can be
// served from LDS: a workgroup (one per compute unit, sixteen waves) keeps a column tile of B -- 32 or 64 bytes of
// every row, up to 5120 rows -- in LDS for its whole life and its waves walk through row panels independently of each
// other, each step reading the rows of one chunk of 64 vectors at the addresses that the operand's LDS-ordered copy
// names.  B is fetched from L2 once per workgroup instead of once per stored vector.
//
// What bounds it: no one unit.  A step is a chunk of 64 vectors and 32 bytes of B: 2 KB of LDS reads (11 clocks of a compute unit, measured), two
// MFMAs (32 clocks of a SIMD), some 21 clocks of its other instructions, and the loads of its record.  A load takes a compute unit 16 clocks
// where a lane asks for 8 or 16 bytes and 4.6 where it asks for 4, whatever the addresses and however many lanes are masked off; with a record
// per chunk that is 20.6 clocks a step of each of four SIMDs, the longest part, half of it for operand rows that a panel of 8 rows does not
// have.  Such panels have two chunks in a record, whose values come with one request and whose codes with one of 4 bytes: 10.3.  More chunks
// cost 65 clocks a step then; the rest is fixed: launch, the fill before the first step, one line of 128 bytes per row of B whatever
// the tile's width (2.4 clocks a row, 4.6 us for 4096 rows; which lanes fetch which pieces makes no difference), and per panel an epilogue of some 130 clocks
// and stores that a wave's later loads queue up behind.
// 16384 x 4096, V = 8, N = 1024, three operands in turn, replayed from a graph (us; a record per chunk and whole turns -> as it is):
//   90 % empty, fp16 / int32            38.1 -> 32.4 / 41.2 -> 34.9     on merged panels, whose requests are full, 37.7 -> 36.6
//   80 % empty, fp16                    54.2 -> 45.5
//   4-bit values and B                  32.3 -> 31.4
//   4096 rows instead of 16384          18.4 -> 16.2
//   2048 columns (64-byte tiles)        21.9 -> 21.5, merged 22.1 -> 21.2
// 10844 x 838, V = 4, L16-R4, N = 128 (short streams): 10.6 -> 8.7; whole calls of the first case 33.2 -> 29.9.
// (8-byte stores by all lanes in the fp16 epilogue: 34.2; rows of B requested two or three steps ahead, sixteen chunks' records
// ahead, ordinary stores instead of streaming ones: within 2 % either way; records of two chunks for full requests: up to 1.05x as long.)
// Against the gather form, on the operand as given / merged: 4096 x 4096, half empty, V = 2, N = 512 42.4 / 20.7 against 104.8 / 28.4 (calls take
// the form of spmm_dense_kernels.hip there, 15.4); 3004 x 2900, 85 % empty, V = 4, unequal panels, 16 x 8 bit 9.8 / 10.2 against 12.6 / 14.3.
// Against a record per chunk and whole turns, the calls that lost: L4-R4, 15240 x 592, V = 8, unequal panels, N = 1024, fp16 26.6 -> 29.0 (its gather 24.4); L16-R8,
// 12822 x 988, V = 2, N = 128 13.1 -> 13.5 (on all columns 10.3).
// Three things keep the LDS reads at their full rate (190 bytes per clock and compute
// unit measured, random rows reach 81):
//   - the LDS image is [row / 16][16-byte segment][row % 16]: a segment of 16 consecutive rows covers all banks once,
//     so a read is free of conflicts when its 16 rows differ modulo 16, whatever the segment;
//   - the copy deals the vectors of a chunk so that the 16 rows read together do differ modulo 16 wherever the pattern
//     has them (mc_resident_pack); the sum over a chunk does not depend on its order;
//   - the segment number is an instruction offset: no address arithmetic per segment.
// The MFMA computes the transposed tile -- dense columns are its rows, panel rows its columns -- so that a lane ends up
// with four neighbouring columns of one output row and stores them directly: no LDS is left for staging, and none is
// needed.
//
// Matrices with more rows of B than fit are cut into equal K-blocks: the workgroup fills one block after the other and
// keeps the accumulators of several panels per wave in registers meanwhile (PPW of them per pass over K).
#include "internal.h"
#include "lds_async.h"
#include "spmm_operand.h"

namespace {

using mcu::v4i;
using mcu::v2i;
using mcu::v4f;
using mcu::lds_v2i;
typedef __attribute__((address_space(1))) const void gptr_t;
typedef __attribute__((address_space(3))) void lptr_t;

// Records (A values and row codes of a chunk, or of two) are requested this many ahead: they come from L2 or beyond, a
// step is far shorter than that latency, and the stores of a finished panel, which a wave's later loads queue up
// behind, take longer still.  (As many as the registers allow.  The last turn's surplus requests go beyond the wave's records,
// at the end of the copy into its padding: resident_requests in internal.h counts them.)
template <int LB, bool R4, int NT, bool HALF> constexpr int ahead = HALF ? (R4 && NT == 4 ? 2 : 4) : (R4 && NT == 4) ? (LB == 16 ? 2 : 4) : RESIDENT_AHEAD;
constexpr int PFB = 3; // (records of one chunk) in the K-blocked form, whose accumulators need the registers

// How a wave walks through its panels.
//   STREAM  all of K is resident: consecutive panels, whose chunks are one stream in memory; the last chunk of a panel
//           is marked
//   SHARED  all of K is resident, few panels: wpp waves share one
//   BLOCKS  K in blocks, the accumulators of PPW panels in registers meanwhile
enum Walk { STREAM, SHARED, BLOCKS };

// NT: 16-byte segments of the column tile.  OUT: type of the result (SlabArgs::float_out), -1: decided at run time.
// HALF: panels of at most 8 rows and one plane (resident_half), two chunks in a record, whose values share one request.
template <int LB, bool R4, int NT, Walk WALK, int OUT, bool HALF>
__global__ __launch_bounds__(1024) void spmm_resident_kernel(SlabArgs a)
{
    constexpr bool L16 = (LB == 16);
    constexpr int NACC = NT * (R4 ? 2 : 1);              // accumulators (v4i) of one panel
    constexpr int SH = R4 ? (LB == 4 ? 8 : 4) : 0;       // scale carried by widened nibbles
    constexpr int PF = ahead<LB, R4, NT, HALF>, PPW = R4 ? 4 : 8;
    constexpr int CH = HALF ? 2 : 1;                     // chunks of a record, each with accumulators of its own
    static_assert(!HALF || (LB != 16 && WALK != BLOCKS), "records of two chunks: one plane, all of B's rows at once");
    static_assert(resident_padding_suffices(PF), "the walk stays inside the copy and its padding");
    static_assert(PF >= 2, "the next record's codes are read before this record's set is refilled");
    const int float_out = OUT < 0 ? a.float_out : OUT;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform: everything derived from it stays in scalar registers
    const int nw = blockDim.x >> 6;
    const int j = lane & 15, g = lane >> 4, ii = (lane & 15) >> 1;
    const unsigned h8 = 8 * (lane & 1);
    // Workgroups go to the eight XCDs round-robin by their linear id.  The column tiles of one panel
    // group all read the same A operands, so they are given ids that are equal modulo 8: one XCD's L2
    // then fetches a group's A operands once for all tiles (and holds all of B, which is small).
    const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int tile = q % a.ntiles, grp = (q / a.ntiles) * 8 + x;
    if (grp >= a.groups) return;
    const int nb0 = tile * (16 * NT);
    const uint8_t *Bb = a.B + nb0;

    const int slots = nw / a.wpp;                         // panel streams of a workgroup
    const int slot = w / a.wpp, k = w % a.wpp;            // this wave: its stream, its share of the stream's one panel (wpp > 1)

    // ---- fill: block b of the tile ---------------------------------------------------------------------
    // Copy instruction u moves 1 KB: four (16 rows, segment) pieces of the image; lane l fetches its segment of row l % 16.
    // Segments beyond the tile or the end of a B row are replaced by segment 0 (never stored), rows beyond K by the last.
    auto fill = [&](int b) {
        const int row0 = b * a.block_rows;
        const int nrows = (a.K - row0 < a.block_rows) ? a.K - row0 : a.block_rows;
        const int units = ((nrows + 15) / 16 * a.nt + 3) / 4;
        for (int u = w; u < units; u += nw) {
            const int piece = u * 4 + g, sg = piece & (a.nt - 1);
            int r = row0 + (piece >> (a.nt == 4 ? 2 : 1)) * 16 + j; // (a.nt is 2 or 4)
            if (r >= a.K) r = a.K - 1;
            const int off = (sg < NT && nb0 + sg * 16 < a.row_bytes) ? sg * 16 : 0;
            __builtin_amdgcn_global_load_lds((gptr_t *)(Bb + (int64_t)r * a.ldb_bytes + off), (lptr_t *)(lds + u * 1024), 16, 0, 0);
        }
    };

    // ---- one chunk ---------------------------------------------------------------------------------------
    // A record of the copy is the codes of one chunk, or of two, followed by the values.  A word of codes: the LDS places (in 16 bytes)
    // of the rows in slots g*16 + ii (low half) and g*16 + 8 + ii.  Two lanes need the same word; with two chunks in a record
    // even lanes load the first chunk's and odd lanes the second's, and hand them over (HANDED; not with tiles of 64 bytes, whose
    // steps have more to do for the VALU: within 2 % there).
    // HALF: the values of both chunks in one request, the first chunk's rows in columns 0 .. 7 of the MFMA's operand, the second's in
    // columns 8 .. 15 (the other columns of each product are not looked at).
    // Records are read through a buffer descriptor: a scalar offset moves from record to record, the lanes' offsets stay.
    // (The descriptor's range check leaves the scalar offset out: what keeps a stream inside the copy is its padding.)
    constexpr bool HANDED = HALF && NT == 2;
    constexpr int WORDS = HALF && !HANDED ? 2 : 1;        // of codes of a record that a lane loads
    constexpr int VALUES = CH * 2 * MC_CHUNK;             // where they begin
    const unsigned lane_r = HANDED ? lane * 4 : (g * 8 + ii) * 4 * CH;
    const int j8 = L16 || HALF ? (j & 7) : j, v_of_j = j8 < a.V ? j8 : 0; // (columns beyond the panel's rows get a copy of row 0)
    constexpr int PIECE = LB == 4 ? 8 : 16;               // bytes of a lane
    const unsigned lane_a = VALUES + (L16 || HALF ? (g * 2 + (j >> 3)) * PIECE * a.V + v_of_j * PIECE : g * PIECE * a.V + v_of_j * PIECE);
    auto records_from = [&](int64_t record) {             // descriptor of the records from this one on
        const int64_t left = (a.nrecs + RESIDENT_PADDING - record) * a.rec_bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.recs) + record * a.rec_bytes, 0, (int)(left < 0x7fffffff ? left : 0x7fffffff),
                                                 0x00020000);
    };
    auto load_rec = [&](__amdgpu_buffer_rsrc_t recs, int offset, v4i &va, int (&r)[WORDS]) { // offset: wave-uniform
        r[0] = __builtin_amdgcn_raw_buffer_load_b32(recs, lane_r, offset, 0);
        if (WORDS == 2) r[WORDS - 1] = __builtin_amdgcn_raw_buffer_load_b32(recs, lane_r + 4, offset, 0);
        if (LB == 4) {
            const v2i x = __builtin_amdgcn_raw_buffer_load_b64(recs, lane_a, offset, 0);
            va = (v4i){x.x, x.y, 0, 0};
        } else {
            va = __builtin_amdgcn_raw_buffer_load_b128(recs, lane_a, offset, 0);
        }
    };
    // the word of codes of chunk h of a record
    auto codes_of = [&](const int (&word)[WORDS], auto H) -> int {
        if (!HANDED) return word[WORDS == 2 ? decltype(H)::value : 0];
        return __builtin_amdgcn_mov_dpp(word[0], decltype(H)::value ? 0xF5 : 0xA0, 0xF, 0xF, true); // quad_perm [1,1,3,3] / [0,0,2,2]
    };
    // the dense operand of a chunk: NT segments of the 64 rows its codes name, transposed
    // (one instruction per address: half of r * 16 + h8.  The kernel has no other LDS, so the image starts at address 0.)
    auto read_b = [&](int r, v4i (&bop)[NT]) {
        unsigned p0, p1;
        asm("v_mad_u32_u16 %0, %1, 16, %2" : "=v"(p0) : "v"(r), "v"(h8));
        asm("v_mad_u32_u16 %0, %1, 16, %2 op_sel:[1,0,0,0]" : "=v"(p1) : "v"(r), "v"(h8));
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const v2i d0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(uintptr_t)(p0 + ct * 256));
            const v2i d1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(uintptr_t)(p1 + ct * 256));
            bop[ct] = (v4i){d0.x, d0.y, d1.x, d1.y};
        }
    };
    auto multiply = [&](v4i (&acc)[NACC], v4i raw, const v4i (&bop)[NT]) {
        const v4i av = mcu::finish_a<LB>(raw);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            if (!R4) {
                acc[ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bop[ct], av, acc[ct], 0, 0, 0);
            } else {
                const v4i msk = {(int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0};
                acc[2 * ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8((bop[ct] << 4) & msk, av, acc[2 * ct], 0, 0, 0);
                acc[2 * ct + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bop[ct] & msk, av, acc[2 * ct + 1], 0, 0, 0);
            }
        }
    };

    // ---- output --------------------------------------------------------------------------------------------
    // Register r of lane (j, g) of accumulator ct is byte column 16 ct + 4 g + r of panel row j (a two-plane A: high plane
    // in j < 8, low plane in j >= 8); a byte column of nibbles is two output columns.  Everything that does not change
    // from panel to panel is worked out here: the epilogue is a good part of a short panel's instructions.
    const int ncols = R4 ? a.row_bytes * 2 : a.row_bytes, es = float_out == 2 ? 2 : 4;
    // HALF: what a panel's rows have in columns 0 .. 7 of segment ct stays there, those of segment ct + 1 go to columns 8 .. 15 (`whole`).
    constexpr int NOUT = HALF ? NACC / 2 : NACC;
    const int jrow = HALF ? (j & 7) : j;
    const int col0 = HALF ? (R4 ? 2 : 1) * (nb0 + 16 * (j >> 3) + 4 * g)
                          : R4 ? 2 * (nb0 + 4 * g) : (float_out == 2 ? nb0 + (g & 1) * 16 + (g >> 1) * 8 : nb0 + 4 * g);
    uint8_t *const out0 = static_cast<uint8_t *>(a.C) + ((int64_t)jrow * a.ldc + col0) * es;
    const int64_t panel_bytes = (int64_t)a.V * a.ldc * es;
    auto finish = [&](v4i s) -> v4i {   // every plane sum is exact in int32 (4-bit B: after its shift); the recombination wraps
        if (R4) s = s >> SH;
        if (L16) {
            v4i lo;
#pragma unroll
            for (int r = 0; r < 4; ++r) lo[r] = __builtin_amdgcn_update_dpp(0, s[r], 0x128, 0xF, 0xF, false); // row_ror:8: lane j + 8
            s = (s << 8) + lo;
        }
        return s;
    };
    // (the product is rounded to fp32 before fp16: the compiler must not fold multiplication and conversion into one instruction)
    auto scaled = [&](v4i s) -> v4f {
        v4f f = {s.x * a.out_scale, s.y * a.out_scale, s.z * a.out_scale, s.w * a.out_scale};
        asm("" : "+v"(f));
        return f;
    };
    // o: out0 of the panel; rows_left: rows of C from the panel's first on (a merged panel may run past the last row)
    constexpr int PER = HALF ? 2 : 1, NSEG = NT / PER;    // segments of an accumulator; steps of that many
    auto store_panel = [&](const v4i (&acc)[NOUT], uint8_t *o, int rows_left) {
        v4i fin[NOUT];
#pragma unroll
        for (int t = 0; t < NOUT; ++t) fin[t] = finish(acc[t]);
        const bool live = jrow < (rows_left < a.V ? rows_left : a.V);
        if constexpr (R4) {
#pragma unroll
            for (int ct = 0; ct < NSEG; ++ct) {
                const v4i e = fin[2 * ct], d = fin[2 * ct + 1];
                const v4i s0 = {e.x, d.x, e.y, d.y}, s1 = {e.z, d.z, e.w, d.w};
                if (float_out == 2) {
                    const mcu::v4h h0 = mcu::to_half4(scaled(s0)), h1 = mcu::to_half4(scaled(s1));
                    if (live && col0 + 32 * PER * ct < ncols) __builtin_nontemporal_store((mcu::v8h){h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w}, reinterpret_cast<mcu::v8h *>(o + ct * 64 * PER));
                } else {
                    const v4i t0 = float_out ? __builtin_bit_cast(v4i, scaled(s0)) : s0, t1 = float_out ? __builtin_bit_cast(v4i, scaled(s1)) : s1;
                    if (live && col0 + 32 * PER * ct < ncols) {
                        __builtin_nontemporal_store(t0, reinterpret_cast<v4i *>(o + ct * 128 * PER));
                        __builtin_nontemporal_store(t1, reinterpret_cast<v4i *>(o + ct * 128 * PER + 16));
                    }
                }
            }
        } else if (HALF && float_out == 2) {
#pragma unroll
            for (int ct = 0; ct < NSEG; ++ct) {
                // the columns of odd lane groups beside those of even ones (stores of 8 bytes by all lanes: 34.2 us where 16 by half of them take 32.5)
                const v2i x = __builtin_bit_cast(v2i, mcu::to_half4(scaled(fin[ct])));
                const auto s0 = __builtin_amdgcn_permlane16_swap((unsigned)x.x, (unsigned)x.x, false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap((unsigned)x.y, (unsigned)x.y, false, false);
                if (live && !(g & 1) && col0 + 32 * ct < ncols)
                    __builtin_nontemporal_store((v4i){(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]}, reinterpret_cast<v4i *>(o + ct * 64));
            }
        } else if (float_out == 2) {
#pragma unroll
            for (int ct = 0; ct < (HALF ? 0 : NT); ct += 2) {
                // lane groups hold columns 4g .. 4g+3 of segments ct and ct + 1; after the exchange of odd groups of the one
                // with even groups of the other, groups 0 .. 3 hold columns 0-7, 16-23, 8-15, 24-31
                v2i x = __builtin_bit_cast(v2i, mcu::to_half4(scaled(fin[ct]))), y = __builtin_bit_cast(v2i, mcu::to_half4(scaled(fin[ct + 1])));
                const auto s0 = __builtin_amdgcn_permlane16_swap((unsigned)x.x, (unsigned)y.x, false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap((unsigned)x.y, (unsigned)y.y, false, false);
                if (live && col0 + 16 * ct < ncols)
                    __builtin_nontemporal_store((v4i){(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]}, reinterpret_cast<v4i *>(o + ct * 32));
            }
        } else {
#pragma unroll
            for (int ct = 0; ct < NSEG; ++ct) {
                const v4i t = float_out ? __builtin_bit_cast(v4i, scaled(fin[ct])) : fin[ct];
                if (live && col0 + 16 * PER * ct < ncols) __builtin_nontemporal_store(t, reinterpret_cast<v4i *>(o + ct * 64 * PER));
            }
        }
    };

    if constexpr (WALK != BLOCKS) {
        int p, p_end;                                     // panels of this wave (SHARED: of the waves that share)
        const int streams = a.groups * slots, at = grp * slots + slot;
        if (WALK == SHARED || a.uniform_chunks > 0) {
            p = (int)((int64_t)a.P * at / streams);
            p_end = (int)((int64_t)a.P * (at + 1) / streams);
        } else {                                          // unequal panels: cut where the chunks are equally many
            p = __builtin_amdgcn_readfirstlane(a.splits[(int)((int64_t)RESIDENT_SPLITS * at / streams)]);
            p_end = __builtin_amdgcn_readfirstlane(a.splits[(int)((int64_t)RESIDENT_SPLITS * (at + 1) / streams)]);
        }
        int c0 = 0, n = 0, before = 0;                    // the wave's chunks: n from c0 on; and one before them if c0 is the second of its record
        if (p < p_end) {
            c0 = a.uniform_chunks > 0 ? p * a.uniform_chunks : __builtin_amdgcn_readfirstlane(a.blk_ptr[p]);
            n = (a.uniform_chunks > 0 ? p_end * a.uniform_chunks : __builtin_amdgcn_readfirstlane(a.blk_ptr[p_end])) - c0;
            if (WALK == SHARED) {                         // (one panel)
                const int all = n;
                c0 += all * k / a.wpp;
                n = all * (k + 1) / a.wpp - all * k / a.wpp;
            }
            if (HALF && n > 0) before = c0 & 1;
            c0 -= before;
            n += before;
        }
        // lane l: which of the chunks 8 l .. 8 l + 7 after chunk c end their panel
        auto load_ends = [&](int c) -> unsigned {
            const int bit = c + 8 * lane, word = (bit >> 5) < a.end_words - 1 ? (bit >> 5) : a.end_words - 2;
            return __builtin_amdgcn_alignbit(a.ends[word + 1], a.ends[word], bit & 31);
        };
        unsigned ends = WALK == STREAM ? load_ends(c0) : 0u;
        const __amdgpu_buffer_rsrc_t recs = records_from(c0 / CH);
        int offset = 0;
        v4i ring_a[PF];
        int ring_r[PF][WORDS];
#pragma unroll
        for (int d = 0; d < PF; ++d) {
            load_rec(recs, offset, ring_a[d], ring_r[d]);
            offset += a.rec_bytes;
        }
        fill(0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                                  // the tile is complete
        v4i acc[CH][NACC];
        auto clear = [&]() {
#pragma unroll
            for (int h = 0; h < CH; ++h)
#pragma unroll
                for (int i = 0; i < NACC; ++i) acc[h][i] = (v4i){0, 0, 0, 0};
        };
        // HALF: a panel's rows are the sum of columns 0 .. 7 of the first chunks' products and 8 .. 15 of the second ones'; two segments
        // come out of it side by side, so that all lanes have something to finish and to store
        auto whole = [&](v4i (&sum)[NOUT]) {
            if constexpr (!HALF) {
#pragma unroll
                for (int i = 0; i < NACC; ++i) sum[i] = acc[0][i];
            } else {
                constexpr int Q = R4 ? 2 : 1;
                const bool low = j < 8;
#pragma unroll
                for (int i = 0; i < NOUT; ++i) {
                    const v4i &x0 = acc[0][i / Q * 2 * Q + i % Q], &x1 = acc[CH - 1][i / Q * 2 * Q + i % Q], &y0 = acc[0][i / Q * 2 * Q + Q + i % Q], &y1 = acc[CH - 1][i / Q * 2 * Q + Q + i % Q];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int mine = low ? x0[r] : y1[r], other = low ? y0[r] : x1[r];
                        sum[i][r] = mine + __builtin_amdgcn_update_dpp(0, other, 0x128, 0xF, 0xF, false); // row_ror:8: lane j + 8
                    }
                }
            }
        };
        clear();
        if (n > 0) {
            // A step multiplies a chunk whose rows of B were requested a step before and requests the rows of the next
            // chunk; after the last chunk of register set d the set is refilled with the record PF further on: compile-time set
            // numbers and unconditional loads, so the compiler's own counted waits are exact.  Every instruction counts:
            // the loop runs whole turns, only the last one ends after the record that is the last -- the first step may belong to the stream
            // before, one at the end to the next, and nothing of theirs is stored (SHARED, where they would spoil the sum: counted) --
            // and a panel's end is one bit test.  (Surplus steps up to a whole turn: 1.05x as long at 16384 x 2048 on merged
            // panels; an exit after every record of every turn 1.05x at 80 % empty, 4096 columns.)
            v4i bop[2][NT];
            p -= WALK == STREAM ? before : 0;
            const int p_first = p + before;
            uint8_t *o = out0 + p * panel_bytes;
            int rows_left = a.rows - p * a.V;
            read_b(codes_of(ring_r[0], std::integral_constant<int, 0>{}), bop[0]);
            // STEPS steps from step i on (Last: as many as are left, in whole records)
            constexpr int STEPS = CH * PF;
            auto turn = [&](int i, auto Last) {
                const unsigned mask = WALK == STREAM ? __builtin_amdgcn_readlane(ends, (i >> 3) & 63) >> (i & 7) : 0u;
                mcu::static_while<STEPS>([&](auto Dc) -> bool {
                    constexpr int c = decltype(Dc)::value, d = c / CH, h = c % CH, next = (c + 1) % STEPS;
                    read_b(codes_of(ring_r[next / CH], std::integral_constant<int, next % CH>{}), bop[(c + 1) & 1]);
                    if (WALK == STREAM || (i + c < n && (c > 0 || i >= before))) multiply(acc[h], ring_a[d], bop[c & 1]);
                    if (h == CH - 1) {
                        load_rec(recs, offset, ring_a[d], ring_r[d]);
                        offset += a.rec_bytes;
                    }
                    if (WALK == STREAM && (mask & (1u << c))) {
                        if ((unsigned)(p - p_first) < (unsigned)(p_end - p_first)) {
                            v4i sum[NOUT];
                            whole(sum);
                            store_panel(sum, o, rows_left);
                        }
                        ++p;
                        o += panel_bytes;
                        rows_left -= a.V;
                        clear();
                    }
                    return !decltype(Last)::value || h < CH - 1 || i + c + 1 < n;
                });
                if (WALK == STREAM && ((i + STEPS) & 511) == 0 && i + STEPS < n) ends = load_ends(c0 + i + STEPS);
            };
            int i = 0;
            for (; i + (WALK == STREAM ? STEPS : 1) <= n; i += STEPS) turn(i, std::false_type{});
            if (WALK == STREAM && i < n) turn(i, std::true_type{});
        }
        if constexpr (WALK == SHARED) {
            // few panels: the waves that share one add up their tiles in LDS (B is no longer needed)
            __syncthreads();
            v4i mine[NOUT];
            whole(mine);
            v4i *part = reinterpret_cast<v4i *>(lds) + (int64_t)w * (NOUT * 64) + lane;
#pragma unroll
            for (int i = 0; i < NOUT; ++i) part[i * 64] = mine[i];
            __syncthreads();
            if (k == 0 && p < p_end) {
                for (int o = 1; o < a.wpp; ++o)
#pragma unroll
                    for (int i = 0; i < NOUT; ++i) mine[i] += part[(o * NOUT + i) * 64];
                store_panel(mine, out0 + p * panel_bytes, a.rows - p * a.V);
            }
        }
    } else {
        // ---- K in blocks: PPW panels per wave and pass --------------------------------------------------------
        // A list of n chunks is walked in max(1, ceil(n / PFB)) groups of PFB steps whose surplus steps do nothing; step d
        // of a group refills register set d with the operands of step d of the next group, of this list or the next one.
        v4i ring_a[PFB];
        int ring_r[PFB][WORDS];
        auto load_chunk = [&](int c, v4i &va, int (&r)[WORDS]) { load_rec(records_from(c), 0, va, r); };
        auto start_ring = [&](int first, int len) {
#pragma unroll
            for (int d = 0; d < PFB; ++d) load_chunk(len > 0 ? first + (d < len ? d : len - 1) : 0, ring_a[d], ring_r[d]);
        };
        auto walk = [&](v4i (&acc)[NACC], int first, int len, int nfirst, int nlen) {
            const int ngroups = len > 0 ? (len + PFB - 1) / PFB : 1;
            for (int gi = 0; gi < ngroups; ++gi) {
                const bool last_group = gi + 1 == ngroups;
                mcu::static_for<PFB>([&](auto Dc) {
                    constexpr int d = decltype(Dc)::value;
                    const int pos = gi * PFB + d;
                    if (pos < len) {
                        v4i bop[NT];
                        read_b(ring_r[d][0], bop);
                        multiply(acc, ring_a[d], bop);
                    }
                    int c;
                    if (!last_group) {
                        const int np = pos + PFB;
                        c = first + (np < len ? np : len - 1);
                    } else {
                        c = nlen > 0 ? nfirst + (d < nlen ? d : nlen - 1) : 0;
                    }
                    load_chunk(c, ring_a[d], ring_r[d]);
                });
            }
        };
        const int in_group = (a.P - grp + a.groups - 1) / a.groups;
        const int rounds = (in_group + nw - 1) / nw;
        for (int t0 = 0; t0 < rounds; t0 += PPW) {
            // panel t of this wave: number grp + groups * (t * waves + w) of the operand's order, the wave running forth and
            // back so that a list sorted by length comes out even; lane t holds its chunk range
            const int t = t0 + lane;
            const int at = grp + a.groups * (t * nw + ((t & 1) ? nw - 1 - w : w));
            const int mine = (lane < PPW && t < rounds && at < a.P) ? (a.order ? a.order[at] : at) : -1;
            v4i acc[PPW][NACC];
#pragma unroll
            for (int i = 0; i < PPW; ++i)
#pragma unroll
                for (int q = 0; q < NACC; ++q) acc[i][q] = (v4i){0, 0, 0, 0};
            for (int b = 0; b < a.nblk; ++b) {
                __syncthreads();                          // nobody reads the block before this one any more
                fill(b);
                const int cb = mine >= 0 ? a.blk_ptr[(int64_t)mine * a.nblk + b] : 0;
                const int ce = mine >= 0 ? a.blk_ptr[(int64_t)mine * a.nblk + b + 1] : 0;
                int first = __builtin_amdgcn_readlane(cb, 0), len = __builtin_amdgcn_readlane(ce, 0) - first;
                start_ring(first, len);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                mcu::static_for<PPW>([&](auto Ic) {
                    constexpr int i = decltype(Ic)::value, in = (i + 1 < PPW) ? i + 1 : i;
                    const int nfirst = __builtin_amdgcn_readlane(cb, in);
                    const int nlen = (i + 1 < PPW) ? __builtin_amdgcn_readlane(ce, in) - nfirst : 0;
                    walk(acc[i], first, len, nfirst, nlen);
                    first = nfirst; len = nlen;
                });
            }
            mcu::static_for<PPW>([&](auto Ic) {
                constexpr int i = decltype(Ic)::value;
                const int p = __builtin_amdgcn_readlane(mine, i);
                if (p >= 0) store_panel(acc[i], out0 + p * panel_bytes, a.rows - p * a.V);
            });
        }
    }
}

template <int LB, bool R4, int NT, Walk WALK, int OUT, bool HALF = false> hipError_t launch_one(const SlabArgs &a, hipStream_t s)
{
    auto kern = spmm_resident_kernel<LB, R4, NT, WALK, OUT, HALF>;
    const int units = ((a.block_rows + 15) / 16 * a.nt + 3) / 4;
    int lds = units * 1024;
    if (WALK == SHARED) { // the tiles of the waves that share a panel meet in the same memory
        const int tiles = a.waves * NT * (R4 ? 2 : 1) * 1024;
        if (tiles > lds) lds = tiles;
    }
    // more than 64 KB of LDS per workgroup has to be asked for
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    // ids of the same panel group are equal modulo 8 (see the kernel): groups are rounded up to a multiple of 8
    dim3 grid((unsigned)((a.groups + 7) / 8 * 8 * a.ntiles)), block(64 * a.waves);
    return launch_kernel(kern, grid, block, lds, s, a);
}

template <int LB, bool R4, int NT, bool HALF> hipError_t launch_walk(const SlabArgs &a, hipStream_t s)
{
    if (a.wpp > 1) return launch_one<LB, R4, NT, SHARED, -1, HALF>(a, s);
    // (the epilogue is part of every step of the unrolled loop: one output type per kernel keeps it small)
    if (a.float_out == 0) return launch_one<LB, R4, NT, STREAM, 0, HALF>(a, s);
    if (a.float_out == 1) return launch_one<LB, R4, NT, STREAM, 1, HALF>(a, s);
    return launch_one<LB, R4, NT, STREAM, 2, HALF>(a, s);
}

template <int LB, bool R4, bool HALF> hipError_t launch_tile(const SlabArgs &a, int nt, hipStream_t s)
{
    if (nt == 4) return launch_walk<LB, R4, 4, HALF>(a, s);
    return launch_walk<LB, R4, 2, HALF>(a, s);
}

template <int LB, bool R4> hipError_t launch_nt(const SlabArgs &a, int nt, hipStream_t s)
{
    if (a.nblk > 1) return launch_one<LB, R4, 2, BLOCKS, -1>(a, s);
    if constexpr (LB != 16) {
        if (resident_half(a.V, LB)) return launch_tile<LB, R4, true>(a, nt, s);
    }
    return launch_tile<LB, R4, false>(a, nt, s);
}

} // namespace

hipError_t launch_spmm_slab(mc_prec prec, const SlabArgs &a, int nt, hipStream_t s)
{
    if (a.P == 0 || a.row_bytes == 0) return hipSuccess;
    switch (prec) {
    case MC_L8R8: return launch_nt<8, false>(a, nt, s);
    case MC_L8R4: return launch_nt<8, true>(a, nt, s);
    case MC_L4R4: return launch_nt<4, true>(a, nt, s);
    case MC_L16R8: return launch_nt<16, false>(a, nt, s);
    case MC_L16R4:
    case MC_L12R4: return launch_nt<16, true>(a, nt, s);
    default: return hipErrorInvalidValue;
    }
}
