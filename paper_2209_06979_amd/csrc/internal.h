// Internal declarations shared by the translation units of the library (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <tuple>

#include "../../include/magicube.h"

// One launch, and its own status.  (<<<>>> puts the configuration aside and takes it back in two more calls of the runtime: 3.1 - 3.3 us of
// host time, 2.85 like this, and the host is what bounds the small calls.)
template <class... P, class... A> inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t s, A &&...args)
{
    std::tuple<P...> values(static_cast<A &&>(args)...);
    return std::apply([&](auto &...v) {
        void *pointers[] = {&v...};
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, pointers, lds, s);
    }, values);
}

struct mc_mat {
    int M, K, V, lhs_bits, P;
    int64_t nvec, nslots, vals_bytes;
    int max_panel_chunks;      // longest panel, in chunks of 64 vectors
    int uniform_chunks;        // chunks of every panel when all panels have the same number (and at least one), else 0
    int uniform_vectors;       // the same of their vectors
    int device;                // HIP device the buffers live on
    int32_t *d_panel_ptr;      // 2*P: chunk-aligned first slot, real end slot
    int32_t *d_row_ptr;        // P+1: interchange row pointers (vector offsets)
    int32_t *d_slot_idx;       // nslots
    uint8_t *d_vals;           // vals_bytes (null for a pattern-only mask)
    // Work items for matrices with very unequal panel lengths (null / 0 otherwise): panels longer
    // than a cap are cut into several items of at most `cap` chunks, so that no single
    // workgroup is left with a tail many times the average.
    int32_t *d_items;          // n_items x 4: panel, first chunk, end chunk, 1 if the panel has several items
    int32_t *d_split_panels;   // n_split: the panels that have several items
    int n_items, n_split;
    int max_item_chunks;       // chunks of the longest item
    // Shares of the SDDMM, one workgroup each: first slot (a multiple of 64), stored vectors, panel, first stored vector's number.  First
    // one per panel, then, where panels are cut (n_cut > 0), that many more: the panels in pieces of at most max_cut_chunks
    // chunks, longest first.
    int32_t *d_shares;         // (P + n_cut) x 4
    int n_cut;
    // LDS-ordered copy of the operand for the SpMM that keeps rows of B resident in LDS (see mc_resident_pack; null when
    // not built: pattern-only masks, operands too sparse or small for it)
    int blk_nt;                // 16-byte segments of a row in the LDS image the codes are made for (2 or 4)
    int block_rows;            // rows of B per K-block
    int nblk;                  // K-blocks
    int64_t blk_chunks;        // chunks over all (panel, block) lists
    int32_t *d_blk_ptr;        // P*nblk + 1
    uint8_t *d_blk_recs;       // records of one or two chunks (and RESIDENT_PADDING of zeros)
    uint32_t *d_blk_ends;      // nblk == 1: a bit per chunk, set where a panel ends (and two words of zeros)
    int32_t *d_blk_src;        // blk_chunks * 64: interchange vector of each slot, -1 for padding
    int32_t *d_order;          // nblk > 1: P panel numbers by falling length (null: all panels have the same number of chunks)
    int32_t *d_splits;         // nblk == 1: RESIDENT_SPLITS + 1 panel numbers, the first that starts at or after i/4096 of the
                               // chunks (null: all panels have the same number of chunks)
    bool blk_valid;            // false once the values were replaced in the panel format only
    // Panels sorted by length class for kernels that give a panel 1, 2, 4 or 8 waves (V = 8 only; null when every
    // panel falls into one class): class b holds the panels of at most 8 << b chunks that class b - 1 does not
    // hold; class 3 also takes what is longer still.
    int32_t *d_class_panels;   // P panel numbers, class after class
    int class_start[5];        // first entry of each class in d_class_panels; [4] = P
    int64_t class_chunks[4];   // chunks of each class's panels
    // Merged copy for the SpMM (null when not built): `merge_group` consecutive panels as one panel of
    // V * merge_group rows at the union of their columns (see mc_merge_host); a complete operand of its own
    // (work items, LDS-ordered copy), never merged again.  Its rows may run past M: launches on it pass M as the
    // number of output rows.
    mc_mat *merged;
    int merge_group;
    int32_t *d_merge_src;      // merged nvec * merge_group: interchange vector of each panel's share, -1 = zeros
    int32_t *d_chunk_vec;      // operands with values: first stored vector of each chunk of the panel format, and how many it has
    bool merged_valid;         // false once the values were replaced in the panel format only
    // The operand with all its columns (null when not built; see spmm_dense_kernels.hip).
    uint8_t *d_dense;
    bool dense_valid;          // false once the values were replaced in other formats only
    bool dense_asked;          // built on request
    mutable std::atomic<bool> dense_read; // a product has read it (new values are written to it if one of the two is true)
};

// Builders that also take V = 16 (4- and 8-bit values): the library's merged copies only.
int mc_layout_query_wide(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, mc_layout *out);
int mc_pack_host_wide(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                      int32_t *panel_ptr, int32_t *slot_idx, void *slot_vals);

// The LDS-ordered copy of an operand (spmm_resident_kernels.hip).  Rows of B are resident in LDS in blocks of block_rows,
// a block's image being [row / 16][segment of 16 bytes][row % 16] with nt segments; the vectors of a (panel, block) list
// (never empty: at least one chunk) are dealt into chunks of 64 such that the 16 rows which one LDS read addresses differ modulo 16 where possible.
//   ptr    P*nblk + 1: first chunk of (panel p, block b) at [p*nblk + b]
//   recs   a record per chunk: 64 codes (uint16: (row / 16)*16*nt + row % 16, the place of the row's segment 0 in 16 bytes; the
//          code of slot s at position (s/16)*16 + (s%8)*2 + (s%16)/8; padded slots name some row of the block), then the values in the layout of a chunk
//          of mc_pack_host's slot_vals.
//          resident_half, one block (one plane of at most 8 rows, half of what a request of the MFMA's operand brings): a record per two
//          chunks, whichever panels they belong to.  Word w of the first chunk's codes is word 2w of the record, that of the second 2w + 1;
//          then the values of both by lane groups: 16 slots of the first, 16 of the second.
//          Zeroed by the caller.
//   src    nchunks*64: interchange vector of each slot, -1 for padding
constexpr int RESIDENT_AHEAD = 8;     // records that a reader has requested ahead of its step, at most
// A reader of n records requests `ahead` of them before its first step and one in every step, and takes whole turns of `ahead`
// steps: this many in all, the surplus ones from what follows (the next reader's records, or the padding).
constexpr int64_t resident_requests(int64_t n, int ahead) { return ahead + (n + ahead - 1) / ahead * ahead; }
// Records of zeros after the copy: what the reader of its last records requests beyond them (most where one record is left
// for the last turn).
constexpr int RESIDENT_PADDING = 2 * RESIDENT_AHEAD - 1;
constexpr bool resident_padding_suffices(int ahead)
{
    for (int n = 0; n <= 4 * ahead; ++n)
        if (resident_requests(n, ahead) > n + RESIDENT_PADDING) return false;
    return true;
}
constexpr bool resident_half(int V, int lhs_bits) { return V <= 8 && lhs_bits <= 8; }
constexpr int resident_rec_chunks(int nblk, int V, int lhs_bits) { return nblk == 1 && resident_half(V, lhs_bits) ? 2 : 1; }
constexpr int RESIDENT_SPLITS = 4096; // an operand with unequal panels has the first panel of every 1/4096 of its chunks listed
struct ResidentLayout { int nt, block_rows, nblk; int64_t nchunks; };
void mc_resident_query(int K, int P, const int32_t *row_ptr, const int32_t *col_idx, ResidentLayout *out);
// bit i of ends: chunk i is the last of its panel (nblk 1 only; (nchunks + 31) / 32 + 2 words)
int mc_resident_pack(int K, int V, int lhs_bits, int P, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                     const ResidentLayout &lay, int32_t *ptr, uint8_t *recs, int32_t *src, uint32_t *ends);

// Chunks of a wave up to which a gathered launch has two of them in flight
constexpr int SPMM_PIPE_CHUNKS = 4;

// One SpMM launch (optionally a batch of problems sharing the sparsity pattern).
struct SpmmArgs {
    const int32_t *panel_ptr;
    const int32_t *slot_idx;
    const uint8_t *vals;
    int64_t vals_batch_stride; // bytes
    const uint8_t *B;
    int64_t ldb_bytes;
    int64_t B_batch_stride;    // bytes
    int row_bytes;             // bytes of one B row that take part (N * bits / 8)
    void *C;                   // int32, float or half (see float_out)
    int64_t ldc;               // elements
    int64_t C_batch_stride;    // elements
    int P, V, batch;
    int rows;                  // rows of C (a merged operand's last panel may run past them); V up to 16
    int float_out;             // 0: int32; 1: float(acc) * out_scale as fp32; 2: the same rounded to fp16
    float out_scale;
    int lhs_unsigned, rhs_unsigned; // 4- and 8-bit operands read as non-negative values
    // optional work items (see mc_mat): null = one unit of work per panel.  Items of a split panel
    // add their int32 results into C with atomics; C's rows of those panels are cleared first.
    const int32_t *items;
    int n_units;               // items, or P
    int stages;                // chunks in flight per wave: 1 or 2 (2 needs short_b)
    int short_b;               // B spans less than 4 GiB, its rows and their length fit 24 bits
    int uniform_chunks;        // > 0: every panel has this many chunks and starts at panel * uniform_chunks * 64 (panel_ptr is not read)
    int ntiles, tile_shift;    // filled by the launcher: column tiles (workgroups) per unit, and their log2 (-1: not a power of two)
    int max_unit_chunks;       // chunks of the longest unit of work (panel or work item)
    // optional: items of a split panel add their int32 results here instead of into C (which may then be float or
    // half): cleared rows [batch][split panel][V][acc_ld], finished by launch_finish_split_rows
    int32_t *acc;
    int acc_ld, n_split;
    long long *trace;          // measurement aid (launch_spmm_phase_probe only): time stamps per wave
};

// One launch of the SpMM that keeps rows of B resident in LDS (see spmm_resident_kernels.hip).
struct SlabArgs {
    const int32_t *blk_ptr;
    const uint8_t *recs;
    const uint32_t *ends;
    int end_words;
    const int32_t *order, *splits; // see mc_mat
    int uniform_chunks;        // > 0: every panel has this many chunks (nblk == 1)
    int rec_bytes;             // bytes of a record
    int64_t nrecs;             // records (RESIDENT_PADDING more follow)
    const uint8_t *B;
    int64_t ldb_bytes;
    int row_bytes, K;
    void *C;
    int64_t ldc;
    int P, V, nblk, block_rows;
    int nt;                    // segments per row of the LDS image (the operand's copy is made for it)
    int rows;                  // rows of C (see SpmmArgs)
    int float_out;
    float out_scale;
    int ntiles;                // column tiles
    int groups;                // panel groups (workgroups per column tile)
    int wpp;                   // waves sharing a panel (its chunks dealt round-robin); above 1 only if every wave has one panel
    int waves;                 // per workgroup, a multiple of wpp
};

// One launch of the SpMM on an operand held with all its columns (see spmm_dense_kernels.hip).
struct DenseArgs {
    const uint8_t *A;          // [block of 16 rows][chunk of 64 columns][plane] fragments of 1 KB: 16 bytes of lane j + 16 g = row j, columns 16 g ..
    int a_bytes;               // its size
    int nrb, nch;              // row blocks, chunks
    const uint8_t *B;
    int64_t ldb_bytes;
    int b_bytes;               // from B's first byte to the end of the last row's part that takes part
    void *C;
    int64_t ldc;
    int rows, cols;            // of C
    int float_out;             // as in SpmmArgs
    float out_scale;
    int tm, tn;                // filled by the launcher: row and column tiles
};
constexpr int DENSE_TILES = 6; // tile shapes of that kernel, numbered from the largest: rows and columns
constexpr int dense_tile_rows(int tile, int planes) { return tile < 2 ? (planes == 1 ? 256 : 128) >> tile : tile == 2 ? 128 : tile == 3 ? 64 : 32; }
constexpr int dense_tile_cols(int tile) { return tile < 2 ? 128 : tile == 5 ? 32 : 64; }
// groups of waves that take turns at its chunks, and the steps that its loop runs as one
constexpr int dense_tile_share(int tile) { return tile == 0 ? 1 : tile == 4 ? 4 : 2; }
constexpr int dense_tile_turn(int tile) { return tile < 4 ? 4 : 8; }
// The copy that kernel reads, written from the panel format.
struct DenseFillArgs {
    const int32_t *panel_ptr, *slot_idx;
    const uint8_t *vals;
    uint8_t *dst;
    int P, V, bits, nch;       // bits 4, 8 or 16
};

struct SddmmArgs {
    const int32_t *shares;     // n_shares x 4 (see mc_mat)
    int n_shares;
    int uniform_vectors;       // > 0: the shares are the panels and each has this many vectors (shares need not be read)
    const int32_t *slot_idx;
    const uint8_t *Q;
    int64_t ldq_bytes, Q_batch_stride;
    const uint8_t *Kmat;
    int64_t ldk_bytes, K_batch_stride;
    int row_bytes;             // Kd * bits / 8
    void *S;                   // int32, float or half (see float_out)
    int64_t S_batch_stride;    // elements
    int float_out;             // 0: int32; 1: float(score) * out_scale as fp32; 2: the same rounded to fp16;
                               // 3: integer codes clamp(rint(score * out_scale)) into a sparse operand's device format
    float out_scale;
    uint8_t *dev_vals;         // float_out 3: the operand's value array, its bytes per batch item, its code width (8 / 16)
    int64_t dev_batch_stride;
    int code_bits;
    int V, batch;
    int lhs_unsigned, rhs_unsigned; // 4- and 8-bit operands read as non-negative values
    int kmat_rows;
};

// Scores + softmax of the attention layer in one kernel (attention_scores_kernels.hip): V = 8, one mask for all heads.
struct ScoresArgs {
    const int32_t *panel_ptr;
    const int32_t *slot_idx;
    const uint8_t *Q, *Km;
    int64_t in_head_stride, in_token_stride; // bytes
    int row_bytes;             // dk * bits / 8, a multiple of 16, at most 256
    float score_scale, inv_s_p;
    uint8_t *dev_vals;         // codes in the device panel format, one block of dev_batch_stride bytes per head
    int64_t dev_batch_stride;
    int P, heads;
    int max_npad;              // longest panel of the mask, padded to whole chunks, in vectors
};

struct SoftmaxArgs {
    const int32_t *row_ptr;
    const int32_t *S;
    void *codes;               // int8 (code_bits 8) or int16 (code_bits 16), interchange order; or null:
    // the codes go straight into the device panel format of a sparse operand (padded slots zeroed)
    const int32_t *panel_ptr;
    uint8_t *dev_vals;
    int64_t dev_batch_stride;  // bytes
    int64_t batch_stride;      // elements (nvec * V)
    float score_scale, inv_s_p;
    int P, V, batch, code_bits;
    int max_panel_chunks;      // longest panel of the mask, in chunks of 64 vectors
    int variant;               // 0: automatic; 1: a workgroup per panel even for short panels; 2: the any-length kernel
};

// One device format that receives an operand's new values.
struct ValuesJob {
    const int32_t *chunk_vec;  // panels: first stored vector and number of vectors of each chunk
    const int32_t *blk_src;    // LDS-ordered copy (else null): the stored vector of each slot, -1 for padding
    const int32_t *merge_src;  // merged copy (else null): the operand's own vector behind each share of a merged vector, -1: zeros
    uint8_t *dst;              // record r's values at r * rec_bytes + head_bytes
    int64_t nchunks;
    int rec_bytes, head_bytes, V, first_block;
    int rec_chunks;            // chunks of a record, 1 or 2 (2: their values by lane groups, see mc_resident_pack)
};
struct ValuesArgs {
    const uint8_t *src;        // interchange order, V values of `bits` per vector
    int V, bits, njobs;
    ValuesJob job[4];
};

// Fused attention (attention_fused.h).  Element (head h, token l, d) of Q, Km, Vm (8- or 4-bit)
// and O (fp32) sits at h*head_stride + l*token_stride + d.
struct AttnArgs {
    // what a wave needs first, in one line of 64 bytes
    const int32_t *panel_ptr;
    const int32_t *slot_idx;
    const int32_t *panel_list;               // the panels of this launch (null: 0 .. P-1)
    int heads, batch;
    int pair_shift, pair_rows;               // set by the launcher: log2 of the (head group, batch item) pairs of a grid row; rows of the grid
    const uint8_t *Km;
    int in_token_stride;                     // bytes of Q, Km, Vm, below 2^24
    int uniform_vectors;                     // > 0: every panel has this many vectors and starts behind the chunks of those before (panel_ptr need not be read)
    int64_t in_head_stride;                  // bytes of Q, Km, Vm
    // (these follow: kernels that do not read uniform_vectors ask for everything from Km to in_batch_stride at once)
    const uint8_t *Q, *Vm;
    int64_t in_batch_stride;                 // between batch items: bytes of Q, Km, Vm
    float *O;                                // fp32, or half when out_f16 is set
    int64_t head_stride, token_stride;       // elements of O
    int64_t batch_stride;
    float score_scale, inv_s_p, out_scale;
    int out_f16;                             // 1: O holds fp16 (the fp32 result rounded to nearest even)
    // head dimensions below the kernel's tile (launch_attention_fused_padded): 16-byte pieces a Q / Kmat / V row
    // really has, and columns of O
    int real_pieces, out_cols;
    // for the launcher: panels, rows of Km and Vm, column indices of this launch's panels
    int P, tokens;
    int64_t index_bytes;
};
static_assert(offsetof(AttnArgs, Q) == 64 && offsetof(AttnArgs, in_batch_stride) == 80, "a line of 64 bytes; one request from Km on");

hipError_t launch_spmm(mc_prec prec, const SpmmArgs &a, int bnb, int waves, hipStream_t s);
// the L8-R8 SpMM (128-byte tiles, 2 waves per panel, two chunks in flight; every panel at most 8 chunks, whole panels,
// B below 4 GiB) with 10 time stamps per wave written to a.trace
hipError_t launch_spmm_phase_probe(const SpmmArgs &a, hipStream_t s);
// nt: segments (16 bytes) of a column tile, 2 or 4, at most a.nt.  Precisions with a 16-bit B are not built.
hipError_t launch_spmm_slab(mc_prec prec, const SlabArgs &a, int nt, hipStream_t s);
// tile: 0 .. DENSE_TILES - 1.  Precisions with a 16-bit B are not built.  A and B span less than 2 GiB each, and
// 8192 rows more of B less than 4 GiB (the kernel's offsets run ahead of the last row, to where its loads return zeros).
hipError_t launch_spmm_dense(mc_prec prec, const DenseArgs &a, int tile, hipStream_t s);
hipError_t launch_dense_fill(const DenseFillArgs &a, hipStream_t s);
hipError_t launch_set_values(ValuesArgs a, hipStream_t s);
// clears the C rows (int32, n columns) of the listed panels
hipError_t launch_zero_rows(int32_t *C, int64_t ldc, int n, int V, const int32_t *panels, int n_panels, hipStream_t s);
hipError_t launch_zero_ints(int32_t *p, int64_t n, hipStream_t s); // n a multiple of 4, p 16-byte aligned
// C rows of the split panels = scale * float(acc rows) (float_out 1: fp32, 2: fp16); acc as in SpmmArgs, n columns
hipError_t launch_finish_split_rows(const int32_t *acc, int n, int n_split, int V, int batch, const int32_t *panels, void *C,
                                    int64_t ldc, int64_t C_batch_stride, int float_out, float scale, hipStream_t s);
// the gather of launch_spmm alone (same tile variant); sink: one int32 per workgroup (P * row tiles)
hipError_t launch_gather_probe(const SpmmArgs &a, int bnb, int waves, int32_t *sink, hipStream_t s);
// `workgroups` x 4 waves x `iters` x 8 MFMAs (16x16x64 i8); sink: workgroups * 256 int32
hipError_t launch_mfma_probe(int workgroups, int iters, int32_t *sink, hipStream_t s);
// waves: 0 = the direct-load kernel; 1, 2, 4, 8 = waves per panel of the LDS-staged kernel
// (used for rows of up to 1024 bytes)
hipError_t launch_sddmm(int bits, const SddmmArgs &a, int waves, hipStream_t s);
hipError_t launch_softmax(const SoftmaxArgs &a, hipStream_t s);
// waves: 2 or 4 per (panel, head); the longest padded panel must not exceed scores_softmax_max_npad(row_bytes, waves)
hipError_t launch_scores_softmax(const ScoresArgs &a, int qkv_bits, int code_bits, int waves, hipStream_t s);
int scores_softmax_max_npad(int row_bytes, int waves);
hipError_t launch_absmax(const float *x, int64_t n, float *result, hipStream_t s);
hipError_t launch_quantize(const float *x, int64_t n, float scale, int bits, uint8_t *q, hipStream_t s);
// Largest inv_s_p for two heads per workgroup by several waves each with 16-bit codes and 8-bit inputs: what is 2^-64 of a row's largest entry has
// no code then (a quarter of a step), and less is all that those kernels may get wrong.
constexpr float FOLDED_MAX_INV_S_P = 0x1p62f;
// dk is 64 or 128.  heads_per_group 2 needs head_stride == dk (token-major layout), rows of at most 64
// bytes and an even head count
hipError_t launch_attention_fused(const AttnArgs &a, int heads_per_group, int waves_per_panel, int p_bits, int qkv_bits,
                                  int dk, hipStream_t s);
// the same kernel for head dimensions below its tile (64 or 128), and up to its tile of 192: one head per workgroup; a.real_pieces, a.out_cols set
hipError_t launch_attention_fused_padded(const AttnArgs &a, int heads_per_group, int waves_per_panel, int p_bits, int qkv_bits, int tile, hipStream_t s);
int attention_fused_max_vectors(); // longest panel (in vectors) the fused kernel accepts
