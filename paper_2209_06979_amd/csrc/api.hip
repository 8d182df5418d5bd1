// C-ABI entry points: argument checks on the host, then kernel launches on the caller's
// stream.  See include/magicube.h for the contract of every function.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <new>
#include <vector>

namespace {

// The calling thread's default choices (all zero = automatic).  A compute call copies either the
// options it was handed or these once, at entry, and never looks at shared state afterwards.
thread_local mc_options t_options = {};

// The SpMM form that holds an operand with all its columns, as spmm_merge asks for it: 0 automatic, -1 never (also where another
// copy is pinned), 1 wherever it exists; then the tile shape, or -1.
int dense_mode(const mc_options &o) { return o.spmm_merge >= MC_SPMM_DENSE ? 1 : o.spmm_merge == 0 ? 0 : -1; }
// Whether options pin part of another form (spmm_stages = 2 and spmm_splitting = 1 are what an SpMM call does by itself).
bool pins_other_form(const mc_options &o) { return o.spmm_stages == 1 || o.spmm_splitting == -1 || o.spmm_slab_waves != 0 || o.spmm_slab_panels != 0; }
int dense_tile(const mc_options &o) { return o.spmm_merge > MC_SPMM_DENSE ? o.spmm_merge - MC_SPMM_DENSE - 1 : -1; }

bool valid_options(const mc_options &o)
{
    const int b = o.spmm_row_tile_bytes, w = o.spmm_waves, d = o.sddmm_waves;
    if (b != 0 && b != 64 && b != 128 && b != 256) return false;
    if (w != 0 && w != 1 && w != 2 && w != 4 && w != 8) return false;
    if (o.spmm_stages < 0 || o.spmm_stages > 2) return false;
    if (o.spmm_splitting < -1 || o.spmm_splitting > 1) return false;
    if (o.spmm_slab < -1 || o.spmm_slab > 1) return false;
    if (o.spmm_slab_waves < 0 || o.spmm_slab_waves > 15) return false;
    if (o.spmm_slab_panels != 0 && o.spmm_slab_panels != 1 && o.spmm_slab_panels != 2 && o.spmm_slab_panels != 4) return false;
    if (d != 0 && d != -1 && d != 1 && d != 2 && d != 4 && d != 8) return false;
    if (o.softmax_variant < 0 || o.softmax_variant > 2) return false;
    if (o.attention_mode < 0 || o.attention_mode > 6) return false;
    const int m = o.spmm_merge;
    if ((m < -1 || m > 1) && m != -MC_SPMM_DENSE && (m < MC_SPMM_DENSE || m > MC_SPMM_DENSE + DENSE_TILES)) return false;
    return true;
}

// The options of one call: the caller's (validated), or the thread's defaults.
int resolve_options(const mc_options *given, mc_options *out)
{
    if (given) {
        if (!valid_options(*given)) return MC_EINVAL;
        *out = *given;
    } else {
        *out = t_options;
    }
    return MC_OK;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int lhs_bits_of(mc_prec p)
{
    switch (p) {
    case MC_L4R4: return 4;
    case MC_L16R8: case MC_L16R16: case MC_L16R4: return 16;
    case MC_L12R4: return 12;
    default: return 8;
    }
}
inline int rhs_bits_of(mc_prec p)
{
    switch (p) {
    case MC_L8R4: case MC_L4R4: case MC_L16R4: case MC_L12R4: return 4;
    case MC_L16R16: return 16;
    default: return 8;
    }
}
inline bool valid_prec(int p) { return p >= MC_L8R8 && p <= MC_L12R4; }

thread_local char g_detail[256] = "";

// Remembers which HIP call failed and why (read back with mc_last_error_detail).
bool hip_ok(hipError_t e, const char *what)
{
    if (e == hipSuccess) return true;
    snprintf(g_detail, sizeof g_detail, "%s: %s", what, hipGetErrorString(e));
    (void)hipGetLastError();
    return false;
}

#define MC_HIP(call)                               \
    do {                                           \
        if (!hip_ok((call), #call)) return MC_EHIP; \
    } while (0)

// Every compute call works on the device the operand was created on: its buffers are not
// addressable from another one.
bool on_device_of(const mc_mat *A)
{
    int cur = -1;
    if (!hip_ok(hipGetDevice(&cur), "hipGetDevice")) return false;
    if (cur != A->device) {
        snprintf(g_detail, sizeof g_detail, "sparse operand lives on device %d, the current device is %d", A->device, cur);
        return false;
    }
    return true;
}

void free_device(mc_mat *A)
{
    if (A->d_panel_ptr) (void)hipFree(A->d_panel_ptr); // (d_row_ptr and d_shares lie behind it)
    if (A->d_slot_idx) (void)hipFree(A->d_slot_idx);
    if (A->d_vals) (void)hipFree(A->d_vals);
    if (A->d_items) (void)hipFree(A->d_items);
    if (A->d_split_panels) (void)hipFree(A->d_split_panels);
    if (A->d_blk_ptr) (void)hipFree(A->d_blk_ptr);
    if (A->d_blk_recs) (void)hipFree(A->d_blk_recs);
    if (A->d_blk_ends) (void)hipFree(A->d_blk_ends);
    if (A->d_blk_src) (void)hipFree(A->d_blk_src);
    if (A->d_order) (void)hipFree(A->d_order);
    if (A->d_splits) (void)hipFree(A->d_splits);
    if (A->d_class_panels) (void)hipFree(A->d_class_panels);
    if (A->d_merge_src) (void)hipFree(A->d_merge_src);
    if (A->d_chunk_vec) (void)hipFree(A->d_chunk_vec);
    if (A->d_dense) (void)hipFree(A->d_dense);
    if (A->merged) {
        free_device(A->merged);
        delete A->merged;
        A->merged = nullptr;
    }
}

// Waves per share of the mask for SDDMM: enough to put about 3200 waves on the chip (4096 of the light ones that stage rows of 32
// bytes, or 64 bytes of nibbles), no more than a share has units of rows (64 of up to 128 bytes, 32 of 256, 16 beyond), and
// so many that no wave has more than 24 units.
// On 70 shapes (V = 2 .. 8, 1 .. 40 chunks per panel, rows of 32 .. 544 bytes) within 5 % of the best count at 66 or more, 5 - 12 %
// off at worst from run to run (profiles/sddmm_waves.txt).
int choose_sddmm_waves(const mc_mat *mask, int shares, int batch, int row_bytes, int bits, const mc_options &o)
{
    if (o.sddmm_waves != 0) return o.sddmm_waves < 0 ? 0 : o.sddmm_waves; // 0 selects the direct-load kernel in launch_sddmm
    const double avg = shares ? (double)(mask->nslots / MC_CHUNK) / shares : 0.0;
    const double units = avg * (row_bytes <= 128 ? 1 : (row_bytes <= 256 ? 2 : 4));
    const double groups = (double)shares * (batch > 0 ? batch : 1);
    const double target = (row_bytes <= 32 || (bits == 4 && row_bytes <= 64)) ? 4096.0 : 3200.0;
    int w = 1;
    // (down to one unit per wave, e.g. 32 panels of 7 chunks: 2.8 us with 4 waves, 2.4 us with 8)
    while (w < 8 && groups * w * 2 <= target && w < units) w *= 2;
    while (w < 8 && units > 24 * w) w *= 2;
    return w;
}

// (the forms with 32-bit lane offsets work out a lane's offset into B with one 24-bit multiplication)
inline bool spmm_short_b(int K, int64_t ldb_bytes, int row_bytes)
{
    return (int64_t)(K - 1) * ldb_bytes + row_bytes < ((int64_t)1 << 32) && K <= (1 << 24) && ldb_bytes < (1 << 24);
}
inline int spmm_stages_for(const mc_options &o, int K, int64_t ldb_bytes, int row_bytes)
{
    return o.spmm_stages != 1 && spmm_short_b(K, ldb_bytes, row_bytes) ? 2 : 1;
}

// The tile (bytes of a row of B) and the waves per panel of a gathered SpMM, and its expected time in us.
struct GatherPlan { int bnb, waves; double us; };

// Workgroups of one gathered launch that the chip holds at once, by LDS (as in SpmmCfg) and wave slots; 0: more than the 64 KB that the
// launcher gives a workgroup.
constexpr int gather_at_once(int bnb, bool r4, int stages, int rows, int waves)
{
    const int tile = rows * ((r4 ? 2 * bnb : bnb) + 4) * 4, lds = waves * std::max(stages * MC_CHUNK * bnb, tile);
    return lds > 65536 ? 0 : 256 * std::min({163840 / lds, 32 / waves, 16});
}
// waves: log2 of the most waves up to 1 << w that fit; n, part: workgroups at once with these, and its reciprocal; of the kernels with one and two
// chunks in flight, and of the one for unsigned operands (one chunk, twelve rows in a tile)
struct GatherAtOnce { struct { int waves; double n, part; } with[2][3][3][4]; };
constexpr GatherAtOnce gather_at_once_all()
{
    GatherAtOnce g = {};
    for (int r4 = 0; r4 < 2; ++r4)
        for (int t = 0; t < 3; ++t)
            for (int kind = 0; kind < 3; ++kind)
                for (int w = 0; w < 4; ++w) {
                    const int stages = kind == 1 ? 2 : 1, rows = kind == 2 ? 12 : 8;
                    int fits = w;
                    while (gather_at_once(64 << t, r4, stages, rows, 1 << fits) == 0) --fits;
                    const double n = gather_at_once(64 << t, r4, stages, rows, 1 << fits);
                    g.with[r4][t][kind][w] = {fits, n, 1.0 / n};
                }
    return g;
}

// Gathered: the tile and the waves with the least expected time.  Launch and start, later with one chunk in flight; the launch that clears rows when panels
// are cut into items; the staged bytes (padded slots and the unused part of a last tile included); the 128-byte lines that rows touch, each tile by
// itself, with rows at all multiples of their length; B, which every XCD fetches for itself, and the operand's values, which every tile reads again; the
// stores; the waves, each by itself and as one of a workgroup's that meet; the chunks of a wave, one after the other, at an even share; those that
// the longest unit's waves still have then; and a last turn of workgroups that leaves compute units idle.  What each costs goes by the width of B, by the
// tile, by whether A has two planes or panels of 16 rows, and for unsigned operands by the width of B.  Fitted (least squares on the logarithm, nothing
// below zero, a variant counting by how near it is to the fastest of its operand) to every tile and number of waves on 7888 drawn operands and on
// 168 of 4096 x 4096 (as at plan_slab), given and merged, three copies of everything in turn; then scaled to the times of the variants picked (the least of
// several expected times is 1 - 3 % too low).
// On 2280 others, given / merged: the time of the variant picked is off by 6.7 / 6.1 % in the median and by 16 % in nine cases of ten, and that variant is
// 2.6 % slower than the fastest of the eight to twelve on average, 0.9 % below 3.6 us or up to 64 panels, by 10 % or less in nine cases of ten, by
// 62 % at worst; unsigned ones 2.0 %.  Without the waves that meet and the one chunk in flight 2.7 / 3.1 %, 1.5 and 1.5 %; without the staged bytes, B and
// the operand's values either, as fitted before, 2.9 / 3.7 %, and off by 9.7 / 8.5 % and 24 %.  (bench.py --variants times them all.)
// As the root of the sum of the squares of what is moved and what a wave waits for 1.9 / 2.1 %, 0.9 and 1.1 %, but a call takes 20 ns longer to decide.
// Still too low where a few long panels gather from all over B: L12-R4, 1184 x 5592, lengths from 1 to 88 chunks, rows of 208 bytes 21 us where 16 are expected.
// lhs_bits: width of the sparse operand's values in this launch (a mask carries none of its own).  items: the launch takes the operand's
// work items.  stages: chunks that the launch may have in flight (SpmmArgs).  unsigned_ops: the kernel for unsigned operands, which has one in flight and no
// tiles of 256 bytes.
GatherPlan plan_gather(const mc_mat *A, int lhs_bits, int row_bytes, int rb, int out_bytes, int batch, bool items, int stages, bool unsigned_ops,
                       const mc_options &o)
{
    struct Cost { double start, items, meet, one, last, byte, line, store, wave, fetch, operand, chunk, late; };
    static const Cost cost[9][3] = {
        {{2.15, 1.62, 0.0413, 0.0244, 0.503, 1.08e-8, 2.31e-8, 6.03e-8, 0.00029, 3.97e-7, 9.79e-9, 0.401, 0.476}, {2.69, 1.3, 0, 0.767, 1.35, 5.44e-8, 1.12e-8, 1.16e-7, 0.000296, 1.11e-7, 0, 0.517, 0.726}},
        {{2.48, 1.04, 0.0851, 0, 1.31, 2.18e-8, 2.25e-8, 3.47e-8, 0.00042, 4.2e-7, 0, 0.488, 0.479}, {3.36, 2.36, 0, 0.0998, 2.46, 5.53e-8, 9.99e-9, 9.06e-8, 0.000322, 2.34e-7, 0, 0.774, 0.769}},
        {{2.18, 1.63, 0.0296, 0, 0.448, 0, 2.17e-8, 2e-8, 0.000321, 4.96e-7, 1.03e-7, 0.39, 0.447}, {2.61, 1.54, 0, 0.364, 1.52, 2.93e-8, 1.02e-8, 1.25e-7, 0.000365, 2.57e-7, 3.77e-8, 0.687, 0.73}},
        {{1.82, 1.99, 0.0507, 0, 0.276, 0, 2.42e-8, 0, 0.000222, 5.21e-7, 1.13e-7, 0.241, 0.31}, {2.05, 1.59, 0, 0.435, 1.09, 1.55e-8, 1.57e-8, 4.6e-8, 0.000305, 4.19e-7, 1.45e-7, 0.38, 0.512}, {2.18, 1.54, 0, 0.853, 3.07, 1.92e-8, 9.76e-9, 1.68e-7, 0.000248, 4.51e-7, 1.49e-7, 0.603, 0.726}},
        {{1.99, 2.34, 0.0923, 0.000366, 0.87, 0, 2.81e-8, 0, 0.000313, 5.73e-7, 5.24e-8, 0.31, 0.322}, {2.19, 2.6, 0.0375, 0.477, 2.4, 1.8e-8, 1.76e-8, 4.53e-8, 0.000301, 5.89e-7, 4.03e-8, 0.555, 0.523}, {2.96, 2.34, 0, 0.713, 4.82, 1.43e-8, 1.38e-8, 6.16e-8, 0.000366, 6.34e-7, 3.8e-8, 0.799, 0.729}},
        {{1.75, 2.51, 0.0553, 0, 0.397, 0, 2.34e-8, 0, 0.000218, 5.92e-7, 9.69e-8, 0.27, 0.331}, {1.93, 2.28, 0, 0.59, 1.16, 1e-8, 1.81e-8, 5.63e-8, 0.000284, 5.34e-7, 9.81e-8, 0.46, 0.566}, {2.26, 2.61, 0, 0.824, 3.16, 1.72e-8, 1.11e-8, 1.12e-7, 0.000247, 4.42e-7, 9.81e-8, 0.666, 0.77}},
        {{1.85, 1.76, 0.0719, 0, 0.393, 0, 2.26e-8, 0, 0.000279, 5.21e-7, 8.87e-8, 0.334, 0.411}, {2.16, 1.44, 0, 0.489, 1.34, 1.06e-8, 1.78e-8, 7.51e-8, 0.000367, 4.33e-7, 8.67e-8, 0.529, 0.618}, {2.34, 0.921, 0, 0.717, 3.3, 2.02e-8, 9.4e-9, 3.05e-7, 0.00034, 3.37e-7, 2.17e-8, 0.844, 0.876}},
        {{2.45, 1.49, 0.0343, 0, 0.323, 1.26e-8, 2.19e-8, 6.71e-8, 0.000287, 4.53e-7, 1.23e-8, 0.436, 0.484}, {3.09, 0.878, 0, 0, 2.12, 3.18e-8, 1.11e-8, 1.23e-7, 0.000282, 2.13e-7, 0, 0.77, 0.792}},
        {{2.09, 1.85, 0.0729, 0, 0.179, 0, 2.43e-8, 0, 0.000183, 5.84e-7, 1.21e-7, 0.322, 0.367}, {2.29, 1.54, 0.0251, 0, 0.615, 1.44e-8, 1.4e-8, 0, 0.000431, 5.8e-7, 1.57e-7, 0.58, 0.603}}
    };
    static constexpr GatherAtOnce at_once = gather_at_once_all();
    const bool r4 = rb == 4, wide = !r4 && !unsigned_ops, two_stages = stages == 2 && !unsigned_ops;
    const Cost *costs = cost[unsigned_ops ? (r4 ? 7 : 8) : rb == 16 ? 6 : (r4 ? 0 : 3) + (lhs_bits > 8 ? 2 : A->V == 16 ? 1 : 0)];
    const double chunks = (double)(A->nslots / MC_CHUNK) * batch, units = (double)(items ? A->n_items : A->P) * batch;
    const double lines = (double)A->nvec * batch, stored = (double)A->M * batch * ((row_bytes << 3 >> (rb == 4 ? 2 : rb == 8 ? 3 : 4)) * out_bytes);
    const double per_unit = chunks / std::max(1.0, units), fetch = (double)A->K * batch * row_bytes, slot_bytes = (lhs_bits == 12 ? 16 : lhs_bits) * A->V / 8.0;
    const int longest = items ? A->max_item_chunks : A->max_panel_chunks;
    // (every call works this out: no division from here on)
    static constexpr double PART[4] = {1.0, 0.5, 0.25, 0.125};
    GatherPlan best = {64, 1, 1e30};
    for (int t = 0; t < (wide ? 3 : 2); ++t) {
        const int bnb = 64 << t;
        if (o.spmm_row_tile_bytes ? std::min(o.spmm_row_tile_bytes, wide ? 256 : 128) != bnb : bnb > 64 && bnb >= 2 * row_bytes) continue;
        const Cost &c = costs[t];
        const int unit = std::min({bnb, 128, row_bytes & -row_bytes}); // rows start at multiples of this, tiles too
        const int tiles = (row_bytes + bnb - 1) >> (6 + t);
        const double groups = std::max(1.0, units * tiles), steps = chunks * tiles;
        const double fixed = c.start + steps * MC_CHUNK * (bnb * c.byte + slot_bytes * c.operand) + lines * (row_bytes + tiles * (128 - unit)) * c.line +
                             stored * c.store + fetch * c.fetch + (items ? c.items : 0.0);
        const double wave = groups * c.wave + c.meet;
        for (int w = 0; w < 4; ++w) {
            if (o.spmm_waves && o.spmm_waves != 1 << w) continue;
            const auto *fits = at_once.with[r4][t][unsigned_ops ? 2 : 0] + w, *two = at_once.with[r4][t][1] + w;
            if (!o.spmm_waves && fits->waves != w) break;
            // two chunks in flight where no wave has more (the launcher's rule, with the waves it then allows)
            const bool pipelined = two_stages && (longest + (1 << two->waves) - 1) >> two->waves <= SPMM_PIPE_CHUNKS;
            if (pipelined) fits = two;
            const double part = PART[fits->waves];
            double us = fixed + (1 << w) * wave + (pipelined ? 0.0 : c.one), share = per_unit * part;
            if (groups > fits->n) {
                const double turns = groups * fits->part;
                const int64_t whole = (int64_t)turns;
                share = steps * fits->part * part;
                if (turns > (double)whole) us += ((double)(whole + 1) - turns) * c.last;
            }
            us += share * c.chunk + std::max(0.0, longest * part - share) * c.late;
            if (us < best.us) best = {bnb, 1 << w, us};
        }
    }
    return best;
}

} // namespace

extern "C" const char *mc_strerror(int status)
{
    switch (status) {
    case MC_OK: return "ok";
    case MC_EINVAL: return "invalid argument";
    case MC_EUNSUPPORTED: return "unsupported precision or operation";
    case MC_EALIGN: return "pointer or leading dimension not 16-byte aligned";
    case MC_EHIP: return "HIP runtime error";
    case MC_ENOMEM: return "out of memory or workspace too small";
    case MC_ERANGE: return "value out of representable range";
    default: return "unknown status";
    }
}

#ifndef MC_SOURCE_ID
#define MC_SOURCE_ID "unidentified"
#endif
extern "C" const char *mc_version(void) { return "0.2+" MC_SOURCE_ID " gfx950"; }

extern "C" const char *mc_last_error_detail(void) { return g_detail; }

extern "C" void mc_options_init(mc_options *o)
{
    if (o) *o = mc_options{};
}

extern "C" int mc_set_thread_options(const mc_options *o)
{
    if (!o) {
        t_options = mc_options{};
        return MC_OK;
    }
    if (!valid_options(*o)) return MC_EINVAL;
    t_options = *o;
    return MC_OK;
}

extern "C" int mc_get_thread_options(mc_options *o)
{
    if (!o) return MC_EINVAL;
    *o = t_options;
    return MC_OK;
}

// The older one-knob setters: each changes one field of the calling thread's defaults.
namespace {
template <class F> int set_field(F &&f)
{
    mc_options o = t_options;
    f(o);
    if (!valid_options(o)) return MC_EINVAL;
    t_options = o;
    return MC_OK;
}
} // namespace

extern "C" int mc_set_spmm_variant(int bytes_per_row_tile, int waves)
{
    return set_field([&](mc_options &o) { o.spmm_row_tile_bytes = bytes_per_row_tile; o.spmm_waves = waves; });
}

extern "C" int mc_set_spmm_stages(int stages)
{
    if (stages != 1 && stages != 2) return MC_EINVAL;
    return set_field([&](mc_options &o) { o.spmm_stages = stages; });
}

extern "C" int mc_set_spmm_splitting(int enable)
{
    return set_field([&](mc_options &o) { o.spmm_splitting = enable ? 0 : -1; });
}

extern "C" int mc_set_spmm_dense(int mode, int tile)
{
    if (mode < -1 || mode > 1 || tile < -1 || tile >= DENSE_TILES) return MC_EINVAL;
    return set_field([&](mc_options &o) {
        if (mode == 1) o.spmm_merge = MC_SPMM_DENSE + 1 + tile;
        else if (o.spmm_merge != -1 && o.spmm_merge != 1) o.spmm_merge = mode == -1 ? -MC_SPMM_DENSE : 0; // (a pin of the other copies stays)
    });
}

extern "C" int mc_set_sddmm_variant(int waves)
{
    // this setter's own convention: -1 automatic, 0 the direct-load kernel
    if (waves < -1) return MC_EINVAL;
    return set_field([&](mc_options &o) { o.sddmm_waves = (waves == -1) ? 0 : (waves == 0 ? -1 : waves); });
}

extern "C" int mc_set_softmax_variant(int variant)
{
    return set_field([&](mc_options &o) { o.softmax_variant = variant; });
}

extern "C" int mc_set_attention_mode(int mode)
{
    return set_field([&](mc_options &o) { o.attention_mode = mode; });
}

namespace {
// Work split of the SpMM that keeps rows of B resident in LDS, and its expected time.
struct SlabPlan { int nt, ntiles, groups, wpp, waves; double us; };

int resident_end_words(const mc_mat *A) { return (int)((A->blk_chunks + 31) / 32 + 2); }
int resident_chunk_bytes(const mc_mat *A) { return 2 * MC_CHUNK + MC_CHUNK * A->V * (A->lhs_bits == 12 ? 16 : A->lhs_bits) / 8; }
int rec_chunks(const mc_mat *A) { return resident_rec_chunks(A->nblk, A->V, A->lhs_bits); }
int resident_rec_bytes(const mc_mat *A) { return rec_chunks(A) * resident_chunk_bytes(A); }
int64_t resident_records(const mc_mat *A) { return (A->blk_chunks + rec_chunks(A) - 1) / rec_chunks(A); }

// Expected times in us of the resident form, fitted (least squares on the relative error, no constant below zero, a byte of a record above it: left
// free, it came out as nothing for records of two chunks and nibbles of B, and of 88 drawn operands of panels of 8 rows seven ran as given, 1.07 - 1.25 times
// as long as merged) to 7888 drawn operands: all precisions, V = 2 / 4 / 8 and merged, 256 .. 16000 rows, 512 .. 8192 columns, rows of B of 32 .. 1024 bytes
// and more, two in five of them of round length, half to 98 % empty, a quarter with panels of unequal length; and to the 168 points of bench.py --sweep, 4096 x 4096, rows
// of 64 to 512 bytes (without them, where all lengths are round, 12 of these calls were 1.03 - 1.27 times as long as with the constants before).  Timed with three copies of everything in turn, as a
// program's operands alternate.  On 2280 others a resident time is off by 6 % in the median and by 14 % in nine cases of ten (in blocks: 12 %, 30 %), and
// the form, tile and waves picked together are 2.9 % slower than the fastest of all on average, by 10 % or less in nine cases of ten, by 81 % at worst
// (with the constants and the copies before: 3.5 %, 12 %, 81 %).
// Resident, all of B's rows at once: launch and start; the fill, a line of B per row, by how many workgroups there are to fill; per
// step of a wave one part per MFMA and one per byte of a chunk's part of a record, both by how many of the sixteen waves have panels; the epilogues; the stores;
// B, which every XCD fetches for itself; waves that share a panel meet; and the steps that the longest panel's waves still have when an even share would be
// done.  By the width of B, by the tile that the copy is made for, and by what a request for operands brings: two planes of 8 rows or fewer, the 8 rows of two chunks, 16 rows.
// In blocks: per block and pass the fill, per step of a wave its own reads, and per panel of a wave a start in each block.
// (A: the operand's layout figures are enough, its copies need not exist yet)
void plan_slab(const mc_mat *A, int row_bytes, bool r4, int out_bytes, const mc_options &o, SlabPlan *pl)
{
    struct Cost { double start, store, meet, fill, mfma, record, panel, late, fetch, uneven; };
    // (two planes of 8 rows; half requests; panels of 16 rows; two planes of fewer rows; each in tiles of 32 and of 64 bytes)
    static const Cost cost[2][4][2] = {
        {{{3.51, 1.03e-7, 0.717, 0.000755, 0.0553, 6.89e-5, 0.00307, 0.0445, 1.31e-6, 0.02}, {3.7, 6.19e-8, 1.05, 0.00104, 0.0562, 4.71e-5, 0.00708, 0.0204, 1.07e-6, 0.0152}},
         {{3.34, 5.43e-8, 0.261, 0.000633, 0.0502, 5.87e-5, 0.00629, 0.038, 1.37e-6, 0.0188}, {3.36, 5.59e-8, 0.884, 0.000968, 0.053, 4.41e-5, 0.00563, 0.027, 1.07e-6, 0.02}},
         {{3.38, 1.04e-7, 0.815, 0.000852, 0.081, 2e-5, 0, 0.0365, 1.2e-6, 0.0176}, {3.71, 1.09e-7, 1.16, 0.00106, 0.0628, 4.71e-5, 0, 0.0365, 9.17e-7, 0.0107}},
         {{3.33, 1.12e-7, 0.402, 0.000676, 0.0616, 7.5e-5, 0.00823, 0.046, 1.33e-6, 0.0128}, {3.62, 0, 0.991, 0.000934, 0.0408, 0.000148, 0.00946, 0.0253, 1.11e-6, 0.0198}}},
        {{{4.39, 3.88e-8, 0.355, 0.000621, 0.0533, 8.35e-5, 0.00178, 0.088, 1.5e-6, 0.0173}, {3.76, 4.69e-8, 1.2, 0.000944, 0.0603, 6.15e-5, 0.00677, 0.104, 1.35e-6, 0.0189}},
         {{3.88, 8.72e-8, 0.471, 0.000478, 0.0645, 2e-5, 0.00405, 0.0797, 1.76e-6, 0.0312}, {3.86, 8.29e-8, 1.02, 0.000662, 0.0641, 2e-5, 0.00585, 0.0876, 1.41e-6, 0.0217}},
         {{4.09, 9.82e-8, 0.586, 0.000625, 0.0848, 2e-5, 0, 0.0919, 1.62e-6, 0}, {3.77, 1.48e-7, 1.29, 0.000839, 0.0686, 2e-5, 0, 0.0881, 1.4e-6, 0.00798}},
         {{3.76, 0, 0.775, 0.00056, 0.0549, 0.000101, 0.0084, 0.082, 1.75e-6, 0.0243}, {3.59, 0, 1.33, 0.000837, 0.0624, 8.89e-5, 0.00898, 0.0974, 1.67e-6, 0.0243}}}
    };
    struct Blocks { double start, pass, row, step, panel; };
    static const Blocks blocks[2] = {{5.0, 4.07, 0.000913, 0.0726, 2.71}, {4.36, 0, 0.000947, 0.19, 3.08}};
    pl->us = 1e30;
    const double lists = (double)A->blk_chunks / A->P;               // chunks of a panel over all its blocks
    const double store = (double)A->M * row_bytes * (r4 ? 2 : 1) * out_bytes;
    for (int nt = A->nblk == 1 ? A->blk_nt : 2; nt >= 2; nt -= 2) {
        SlabPlan q;
        q.nt = nt;
        q.ntiles = (row_bytes + 16 * nt - 1) / (16 * nt);
        // one workgroup per compute unit; the tiles of a group share an XCD (32 compute units)
        q.groups = 8 * std::max(1, 32 / q.ntiles);
        if (q.groups > A->P) q.groups = A->P;
        const int in_group = (A->P + q.groups - 1) / q.groups;
        q.waves = o.spmm_slab_waves ? o.spmm_slab_waves : 16;
        q.wpp = 1;
        if (A->nblk == 1 && !o.spmm_slab_waves)
            while (q.wpp < 8 && in_group * q.wpp * 2 <= q.waves && q.wpp * 2 <= lists) q.wpp *= 2;
        const int rounds = ((q.groups + 7) / 8 * q.ntiles + 31) / 32;
        const int passes = A->nblk == 1 ? 1 : (in_group + q.waves * (r4 ? 4 : 8) - 1) / (q.waves * (r4 ? 4 : 8));
        // steps of the busiest wave: whole panels, or, where panels are unequal, a fair share
        double steps;
        if (A->nblk > 1) steps = (in_group + q.waves - 1) / q.waves * std::max(lists, 2.0 * A->nblk);
        else if (A->uniform_chunks && in_group >= q.waves) steps = (in_group + q.waves - 1) / q.waves * lists;
        else if (in_group >= q.waves) steps = in_group * lists / q.waves;
        else steps = lists / q.wpp;
        const int mfma = nt * (r4 ? 2 : 1);
        if (A->nblk == 1) {
            const double filling = std::min(256, q.groups * q.ntiles) / 256.0, busy = std::min(1.0, (double)in_group * q.wpp / q.waves);
            const double late = std::max(0.0, (double)A->max_panel_chunks / q.wpp - steps);
            const Cost &c = cost[r4][resident_half(A->V, A->lhs_bits) ? 1 : A->lhs_bits <= 8 ? 2 : A->V == 8 ? 0 : 3][A->blk_nt == 4];
            q.us = c.start + store * c.store + (double)A->K * row_bytes * c.fetch + (q.wpp > 1 ? c.meet : 0.0) +
                   rounds * (A->block_rows * filling * c.fill + steps * busy * mfma * (c.mfma + (A->uniform_chunks ? 0.0 : c.uneven)) +
                             steps * busy * filling * resident_chunk_bytes(A) * c.record +
                             in_group * mfma * c.panel + late * c.late);
        } else {
            const Blocks &c = blocks[r4];
            q.us = c.start + store * 3e-7 + rounds * (passes * A->nblk * (c.pass + A->block_rows * c.row) + steps * c.step +
                                                      (in_group + q.waves - 1) / q.waves * c.panel);
        }
        if (q.us < pl->us) *pl = q;
    }
}

// Whether a gathered call takes the operand's work items (out_mode as in spmm_impl)
bool takes_items(const mc_mat *A, int out_mode, const mc_options &o) { return A->n_items && o.spmm_splitting != -1 && out_mode == 0; }

// Gathered, with signed operands, int32 results and B's rows one after the other
double gather_us(const mc_mat *A, int row_bytes, int rb, const mc_options &o)
{
    return plan_gather(A, A->lhs_bits, row_bytes, rb, 4, 1, takes_items(A, 0, o), spmm_stages_for(o, A->K, row_bytes, row_bytes), false, o).us;
}

// With all columns: the tile shape and the expected time.
struct DensePlan { int tile; double us; };

int64_t dense_bytes(int M, int K, int bits) { return (int64_t)((M + 15) / 16) * ((K + MC_CHUNK - 1) / MC_CHUNK) * 1024 * (bits > 8 ? 2 : 1); }

bool dense_possible(int M, int K, int bits)
{
    return M > 0 && K > 0 && bits != 0 && dense_bytes(M, K, bits) <= INT32_MAX;
}

// Expected time: launch and start; then the longer of a workgroup's steps one after the other (as many turns as its compute unit cannot
// hold of them at once) and of all steps of a compute unit at the rate at which it takes in operands, each with what starting and
// finishing a tile costs; and the stores.  Fitted per tile, planes and width of B to 900 drawn operands, three copies in turn (256 .. 16000
// rows, 512 .. 8192 columns, rows of B of 32 .. 1024 bytes): off by 2 - 7 % in the median and by 6 - 24 % in nine cases of ten; the tile
// picked is 0.5 % slower than the best on average, 25 % at worst, and where the time expected is 3 % below the measured one of the other
// forms (237 of the 900) the call is 1.2 times as fast in the mean.
DensePlan plan_dense(int M, int K, int bits, int row_bytes, bool r4, int out_bytes, int only = -1)
{
    struct Cost { double start, step, stream, store, tile; };
    static const Cost cost[2][2][DENSE_TILES] =
       {{{{1.54e-06, 0.328, 0.562, 1.2e-07, 6.31}, {2.92e-08, 0.424, 0.1, 2.1e-07, 5.62}, {3.45, 0.308, 0.404, 1.5e-07, 0}, {2.91, 0.219, 0.302, 7.4e-08, 0.155}, {1.58, 0.379, 0.401, 5.6e-07, 1.03}, {2.16, 0.0648, 0.176, 2.1e-09, 1.11}},
         {{2.63, 0.357, 0.569, 1e-07, 4.22}, {5.04e-07, 0.443, 0.603, 9.6e-08, 6.34}, {3.41, 0.258, 0.377, 1.3e-07, 0.677}, {2.96, 0.197, 0.26, 1.2e-07, 0.695}, {1.97, 0.297, 0.359, 3.5e-07, 1.87}, {3.05, 0.119, 0.145, 3.4e-08, 0}}},
        {{{3.16, 0.355, 0.527, 9.1e-08, 1.69}, {1.15, 0.417, 0.57, 7.1e-09, 4.42}, {0.703, 0.467, 0.225, 2e-07, 3.61}, {3.16, 0.283, 0.405, 2.1e-07, 0.311}, {1.81, 0.468, 0.512, 3.9e-07, 1.82}, {2.76, 0.16, 0.22, 7.6e-08, 0}},
         {{0.314, 0.415, 0.542, 7.7e-08, 4.75}, {1.02, 0.513, 0.0347, 1.4e-07, 4.19}, {1.36, 0.437, 0.514, 1.2e-07, 3.63}, {3.65, 0.285, 0.354, 2e-07, 0.353}, {2.12, 0.412, 0.479, 6.1e-07, 2.05}, {3.09, 0.157, 0.184, 4e-07, 0}}}};
    const int planes = bits > 8 ? 2 : 1, cols = row_bytes * (r4 ? 2 : 1), chunks = (K + MC_CHUNK - 1) / MC_CHUNK;
    DensePlan best = {-1, 1e30};
    for (int tile = 0; tile < DENSE_TILES; ++tile) {
        if (only >= 0 && tile != only) continue;
        const Cost &c = cost[planes - 1][r4][tile];
        const int rows = dense_tile_rows(tile, planes), turn = dense_tile_turn(tile), share = dense_tile_share(tile);
        const int at_once = tile == 5 ? 4 : tile == 3 || (tile == 2 && planes == 1) ? 2 : 1; // workgroups of a compute unit
        const int steps = ((chunks + share - 1) / share + turn - 1) / turn * turn;
        const int64_t tiles = (int64_t)((M + rows - 1) / rows) * ((cols + dense_tile_cols(tile) - 1) / dense_tile_cols(tile));
        const double turns = (double)((tiles + 256 * at_once - 1) / (256 * at_once)), mean = tiles / 256.0, most = (double)((tiles + 255) / 256);
        const double us = c.start + std::max(turns * (steps * c.step + c.tile), 0.5 * (mean + most) * (steps * c.stream + c.tile / at_once)) +
                          (double)M * cols * out_bytes * c.store;
        if (us < best.us) best = {tile, us};
    }
    return best;
}

// Which of an operand and its merged copy (null: none) get an LDS-ordered copy.  One does where its form is expected to be faster than either gather
// by a twentieth, an expected time's own error, for some width of B, rows of 128 to 1024 bytes.  Where both do, the given operand's is built if it is
// expected to be faster than merged by 15 % for some width, and the merged copy's unless that one is and nothing is gained beside it, a twentieth for
// some width.  Both are decided at once: with the merged copy decided first, giving way to what the given operand could have, that one failed its
// own test at times, and of 10731 operands of 4- and 8-bit values 253 had neither (14952 x 531, V = 8, L4-R4 gathered where it had run resident).
// Of 2280 drawn operands 1225 have one copy then, 34 both, and of 518 with panels of 8 rows and one plane 14 run more than 5 % behind
// their merged resident form (with the rule and the constants before 1338, 70 and 34).
// (2 % over the gathers: operands of 1000 to 2000 rows had the copy for what is no gain, mc_mat_create 1.16 instead of 0.78 ms at
// 2048 x 2048, 90 % empty, and new values to write there.)
struct ResidentCopies { bool given, merged; };
ResidentCopies resident_worth_building(const mc_mat *A, const mc_mat *merged)
{
    const mc_options automatic = {};
    const mc_mat *const of[2] = {A, merged};
    bool worth[2] = {}, beside[2] = {};                   // (a copy beside the other one)
    for (int row_bytes : {1024, 512, 256, 128}) {
        for (int r4 = (A->lhs_bits == 4); r4 < 2; ++r4) {
            double gather = 1e30, us[2] = {1e30, 1e30};
            for (int i = 0; i < 2; ++i) {
                if (!of[i]) continue;
                gather = std::min(gather, gather_us(of[i], row_bytes, r4 ? 4 : 8, automatic));
                if (!of[i]->blk_chunks) continue;
                SlabPlan pl;
                plan_slab(of[i], row_bytes, r4, 4, automatic, &pl);
                us[i] = pl.us;
            }
            for (int i = 0; i < 2; ++i) {
                worth[i] |= us[i] < 0.95 * gather;
                beside[i] |= us[i] < std::min(0.95 * gather, (i == 0 ? 0.85 : 0.95) * us[1 - i]);
            }
        }
    }
    if (!worth[0] || !worth[1]) return {worth[0], worth[1]};
    return {beside[0], !beside[0] || beside[1]};
}

} // namespace

namespace {
// Whether the copy with all columns is built: the form is expected to be the fastest for wide rows of B, or for rows of two lines.
bool dense_worth_building(const mc_mat *A)
{
    const mc_options automatic = {};
    for (int row_bytes : {1024, 512, 256, 128}) {
        for (int r4 = (A->lhs_bits == 4); r4 < 2; ++r4) {
            double best = 1e30;
            for (const mc_mat *X : {A, (const mc_mat *)A->merged}) {
                if (!X) continue;
                best = std::min(best, gather_us(X, row_bytes, r4 ? 4 : 8, automatic));
                if (!X->blk_chunks) continue;
                SlabPlan pl;
                plan_slab(X, row_bytes, r4, 4, automatic, &pl);
                best = std::min(best, pl.us);
            }
            if (plan_dense(A->M, A->K, A->lhs_bits, row_bytes, r4, 4).us < 0.95 * best) return true;
        }
    }
    return false;
}

// Appends the panels in pieces to `shares` (see mc_mat) if any is cut; returns their number.
int cut_shares(const mc_mat *A, const int32_t *row_ptr, const int32_t *panel_ptr, std::vector<int32_t> &shares)
{
    // Pieces of the average panel's chunks; of fewer than 256 panels, of as few (two at least) as make 512 of them.  Whole calls, us, against
    // pieces of 8 chunks at least, 256 of them at least:  L16-R16, 2000 x 3100, V = 4, 90 % empty, unequal (sigma = 0.5), Kd = 200
    // 9.5 -> 8.6;  L8-R8, 4096 x 4096, V = 8, 90 %, unequal (1), Kd = 256 7.2 -> 6.6;  512 x 4096, half empty 5.6 -> 4.5.  Equal panels of
    // 256 and more are better whole (681 of 4 chunks 4.9, halved 5.4) or gain nothing to rely on (512 of 7 chunks 6.0,
    // in pieces of 4 / 3 / 2 chunks 6.0 / 5.7 / 6.3).
    const double total = (double)(A->nslots / MC_CHUNK);
    const int cap = std::max(2, (int)std::ceil(A->P >= 256 ? total / A->P : std::min(total / A->P, total / 512)));
    if (A->max_panel_chunks <= cap) return 0;
    std::vector<std::vector<int32_t>> by_length((size_t)cap + 1); // longest first: they start first and do not form the tail
    for (int p = 0; p < A->P; ++p) {
        const int n = row_ptr[p + 1] - row_ptr[p], c = (n + MC_CHUNK - 1) / MC_CHUNK, pieces = (c + cap - 1) / cap, per = pieces ? (c + pieces - 1) / pieces : 0;
        for (int b = 0; b < c; b += per) {
            const int e = std::min(c, b + per);
            auto &to = by_length[(size_t)(e - b)];
            to.insert(to.end(), {panel_ptr[2 * (size_t)p] + b * MC_CHUNK, std::min(n, e * MC_CHUNK) - b * MC_CHUNK, p, row_ptr[p] + b * MC_CHUNK});
        }
    }
    const size_t before = shares.size();
    for (size_t l = by_length.size(); l-- > 0;) shares.insert(shares.end(), by_length[l].begin(), by_length[l].end());
    return (int)((shares.size() - before) / 4);
}

// The shares of one SDDMM launch (cut: panels of unequal length in pieces)
void take_shares(const mc_mat *A, bool cut, SddmmArgs *a)
{
    const bool pieces = cut && A->n_cut > 0;
    a->shares = A->d_shares + (pieces ? 4 * (int64_t)A->P : 0);
    a->n_shares = pieces ? A->n_cut : A->P;
    a->uniform_vectors = pieces ? 0 : A->uniform_vectors;
    a->kmat_rows = A->K;
}

DenseFillArgs dense_fill_args(const mc_mat *A)
{
    DenseFillArgs f = {};
    f.panel_ptr = A->d_panel_ptr; f.slot_idx = A->d_slot_idx; f.vals = A->d_vals; f.dst = A->d_dense;
    f.P = A->P; f.V = A->V; f.bits = A->lhs_bits == 12 ? 16 : A->lhs_bits; f.nch = (A->K + MC_CHUNK - 1) / MC_CHUNK;
    return f;
}

// Whether mc_mat_create builds the merged copy (lay: the operand, ml: its merged form).  The copy holds
// ml.nvec * rows values; which of the two a call uses is decided per call (spmm_form).
bool merged_worth_building(const mc_layout &lay, const mc_merged_layout &ml) { return ml.nvec <= lay.nvec; }

// The layout of A's LDS-ordered copy, whether it is built or not (no chunks: it cannot be)
void resident_layout(mc_mat *A, const int32_t *row_ptr, const int32_t *col_idx)
{
    ResidentLayout rl;
    mc_resident_query(A->K, A->P, row_ptr, col_idx, &rl);
    if (rl.nchunks * MC_CHUNK > INT32_MAX) return;
    A->blk_nt = rl.nt; A->block_rows = rl.block_rows; A->nblk = rl.nblk; A->blk_chunks = rl.nchunks;
}

// of: the operand whose merged copy this is (V up to 16, never merged again), else null; of_resident: whether that one gets an LDS-ordered copy
int mat_create_impl(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                    void *stream, const mc_mat *of, bool *of_resident, mc_mat **out)
{
    if (!out) return MC_EINVAL;
    *out = nullptr;
    if (!values) lhs_bits = 0;
    if (!of && V == 16) return MC_EINVAL;
    mc_layout lay;
    int rc = mc_layout_query_wide(M, K, V, lhs_bits, row_ptr, &lay);
    if (rc != MC_OK) return rc;

    std::vector<int32_t> panel_ptr, slot_idx;
    std::vector<uint8_t> vals;
    try {
        panel_ptr.resize((size_t)2 * lay.P);
        slot_idx.resize((size_t)lay.nslots);
        vals.resize((size_t)lay.vals_bytes);
    } catch (const std::bad_alloc &) {
        return MC_ENOMEM;
    }
    rc = mc_pack_host_wide(M, K, V, lhs_bits, row_ptr, col_idx, values, panel_ptr.data(), slot_idx.data(),
                           vals.empty() ? nullptr : vals.data());
    if (rc != MC_OK) return rc;

    mc_mat *A = new (std::nothrow) mc_mat();
    if (!A) return MC_ENOMEM;
    A->M = M; A->K = K; A->V = V; A->lhs_bits = lhs_bits; A->P = lay.P;
    A->nvec = lay.nvec; A->nslots = lay.nslots; A->vals_bytes = lay.vals_bytes;
    A->max_panel_chunks = 0;
    int min_panel_chunks = INT32_MAX;
    A->uniform_vectors = lay.P > 0 ? row_ptr[1] - row_ptr[0] : 0;
    for (int p = 0; p < lay.P; ++p) {
        if (row_ptr[p + 1] - row_ptr[p] != A->uniform_vectors) A->uniform_vectors = 0;
        const int c = (row_ptr[p + 1] - row_ptr[p] + MC_CHUNK - 1) / MC_CHUNK;
        if (c > A->max_panel_chunks) A->max_panel_chunks = c;
        if (c < min_panel_chunks) min_panel_chunks = c;
    }
    A->uniform_chunks = (lay.P > 0 && min_panel_chunks == A->max_panel_chunks && min_panel_chunks > 0) ? min_panel_chunks : 0;
    A->d_panel_ptr = A->d_row_ptr = A->d_slot_idx = nullptr;
    A->d_vals = nullptr;
    A->d_items = A->d_split_panels = nullptr;
    A->n_items = A->n_split = 0;
    A->d_shares = nullptr; A->n_cut = 0;
    A->max_item_chunks = 0;
    A->blk_nt = A->block_rows = A->nblk = 0; A->blk_chunks = 0; A->blk_valid = false; A->d_order = A->d_splits = nullptr;
    A->d_blk_ptr = nullptr; A->d_blk_recs = nullptr; A->d_blk_ends = nullptr; A->d_blk_src = nullptr;
    A->d_class_panels = nullptr;
    A->merged = nullptr; A->merge_group = 0; A->d_merge_src = nullptr; A->d_chunk_vec = nullptr; A->merged_valid = false;
    A->d_dense = nullptr; A->dense_valid = false; A->dense_read = false; A->dense_asked = dense_mode(t_options) == 1;
    // Length classes of the panels (V = 8: the attention kernel gives a panel 1, 2, 4 or 8 waves)
    std::vector<int32_t> class_panels;
    for (int b = 0; b <= 4; ++b) A->class_start[b] = 0;
    for (int b = 0; b < 4; ++b) A->class_chunks[b] = 0;
    if (V == 8 && lay.P > 0) {
        auto chunks_of = [&](int p) { return (row_ptr[p + 1] - row_ptr[p] + MC_CHUNK - 1) / MC_CHUNK; };
        auto class_of = [&](int p) {
            const int c = chunks_of(p);
            return c <= 8 ? 0 : (c <= 16 ? 1 : (c <= 32 ? 2 : 3));
        };
        int count[4] = {0, 0, 0, 0};
        for (int p = 0; p < lay.P; ++p) {
            ++count[class_of(p)];
            A->class_chunks[class_of(p)] += chunks_of(p);
        }
        if ((count[0] > 0) + (count[1] > 0) + (count[2] > 0) + (count[3] > 0) > 1) {
            try {
                class_panels.resize((size_t)lay.P);
            } catch (const std::bad_alloc &) {
                delete A;
                return MC_ENOMEM;
            }
            int next[4];
            for (int b = 0, at = 0; b < 4; ++b) { A->class_start[b] = next[b] = at; at += count[b]; }
            A->class_start[4] = lay.P;
            for (int p = 0; p < lay.P; ++p) class_panels[(size_t)next[class_of(p)]++] = p;
        }
    }
    // Work items: only when the longest panel is far above the average; a panel is then cut into
    // pieces of at most `cap` chunks (cap = three times the average, at least 8: smaller pieces
    // balance better but cost the SpMM more in atomics than they gain; measured).
    std::vector<int32_t> items, split_panels;
    {
        const double avg = lay.P ? (double)(lay.nslots / MC_CHUNK) / lay.P : 0.0;
        // A pattern-only mask (its items serve the last SpMM of the attention layer's pipeline, on request) is cut
        // as soon as a panel exceeds the average rounded up to 8 chunks.
        // With fewer than 256 panels the pieces also get short enough to make 256 of them.
        const bool mask_only = (lhs_bits == 0);
        double piece = (mask_only ? 1.0 : 3.0) * avg;
        if (mask_only && lay.P < 256) piece = std::min(piece, (double)(lay.nslots / MC_CHUNK) / 256.0);
        const int cap = std::max(8, (int)std::ceil(piece));
        if (A->max_panel_chunks > (mask_only ? cap : 2 * cap)) {
            try {
                for (int p = 0; p < lay.P; ++p) {
                    const int c = (row_ptr[p + 1] - row_ptr[p] + MC_CHUNK - 1) / MC_CHUNK;
                    const int pieces = (c + cap - 1) / cap;
                    if (pieces > 1) split_panels.push_back(p);
                    if (pieces <= 1) {
                        items.insert(items.end(), {p, 0, c, 0});
                    } else {
                        const int per = (c + pieces - 1) / pieces;
                        // (fourth field: 1 + the panel's position in split_panels)
                        for (int b = 0; b < c; b += per) items.insert(items.end(), {p, b, std::min(c, b + per), (int)split_panels.size()});
                    }
                }
                // longest first: workgroups start in this order, so the long items do not form the tail
                const size_t ni = items.size() / 4;
                std::vector<size_t> order(ni);
                for (size_t i = 0; i < ni; ++i) order[i] = i;
                std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) {
                    return items[4 * x + 2] - items[4 * x + 1] > items[4 * y + 2] - items[4 * y + 1];
                });
                std::vector<int32_t> sorted(items.size());
                for (size_t i = 0; i < ni; ++i) std::copy(items.begin() + 4 * order[i], items.begin() + 4 * order[i] + 4, sorted.begin() + 4 * i);
                items.swap(sorted);
            } catch (const std::bad_alloc &) {
                delete A;
                return MC_ENOMEM;
            }
            A->n_items = (int)(items.size() / 4);
            A->n_split = (int)split_panels.size();
            A->max_item_chunks = 0;
            for (size_t i = 0; i < items.size(); i += 4) A->max_item_chunks = std::max(A->max_item_chunks, items[i + 2] - items[i + 1]);
        }
    }
    // Shares of the SDDMM: every share writes its own outputs, nothing is added up
    std::vector<int32_t> shares;
    if (!of && lay.P > 0) {
        try {
            shares.reserve((size_t)lay.P * 4);
            for (int p = 0; p < lay.P; ++p) shares.insert(shares.end(), {panel_ptr[2 * (size_t)p], row_ptr[p + 1] - row_ptr[p], p, row_ptr[p]});
            A->n_cut = cut_shares(A, row_ptr, panel_ptr.data(), shares);
        } catch (const std::bad_alloc &) {
            delete A;
            return MC_ENOMEM;
        }
    }
    // Merged copy for the SpMM: panels of fewer rows than the matrix unit takes share one panel of 16 rows (4- and
    // 8-bit values) or 8 rows (two byte planes), see mc_merge_host.  Not for operands without vectors, and not
    // when the thread's options rule it out.
    std::vector<int32_t> m_src;
    bool resident = false;                                // (decided with the merged copy's, where there is one)
    if (lhs_bits != 0 && lay.nvec > 0 && t_options.spmm_slab != -1) resident_layout(A, row_ptr, col_idx);
    if (!of && lhs_bits != 0 && lay.nvec > 0 && t_options.spmm_merge != -1) {
        const int rows = (lhs_bits == 4 || lhs_bits == 8) ? 16 : 8, group = rows / V;
        mc_merged_layout ml;
        if (group >= 2 && mc_merged_query(M, K, V, lhs_bits, row_ptr, col_idx, group, &ml) == MC_OK && ml.nvec > 0 &&
            (t_options.spmm_merge == 1 || t_options.spmm_merge >= MC_SPMM_DENSE || merged_worth_building(lay, ml))) {
            std::vector<int32_t> m_row_ptr, m_col_idx;
            std::vector<uint8_t> m_values;
            const int64_t vb = (int64_t)V * (lhs_bits == 12 ? 16 : lhs_bits) / 8;
            try {
                m_row_ptr.resize((size_t)ml.P + 1);
                m_col_idx.resize((size_t)ml.nvec);
                m_values.resize((size_t)(ml.nvec * group * vb));
                m_src.resize((size_t)(ml.nvec * group));
            } catch (const std::bad_alloc &) {
                free_device(A);
                delete A;
                return MC_ENOMEM;
            }
            rc = mc_merge_host(M, K, V, lhs_bits, row_ptr, col_idx, values, group, m_row_ptr.data(), m_col_idx.data(), m_values.data(),
                               m_src.data());
            if (rc == MC_OK)
                rc = mat_create_impl(ml.P * rows, K, rows, lhs_bits, m_row_ptr.data(), m_col_idx.data(), m_values.data(), stream, A,
                                     &resident, &A->merged);
            if (rc != MC_OK) {
                free_device(A);
                delete A;
                return rc;
            }
            A->merge_group = group;
        }
    }
    // LDS-ordered copy for the SpMM that keeps rows of B resident in LDS, where that form is expected to be the fastest one
    // for some width of B (the merged copy's forms included), unless the thread's options rule that kernel out (1: built whatever the shape, so that the
    // form can be forced).
    std::vector<int32_t> blk_ptr, blk_src, order, splits;
    std::vector<uint8_t> blk_recs;
    std::vector<uint32_t> blk_ends;
    if (lhs_bits != 0 && lay.nvec > 0 && t_options.spmm_slab != -1) {
        const ResidentLayout rl = {A->blk_nt, A->block_rows, A->nblk, A->blk_chunks};
        if (of) {
            const ResidentCopies copies = resident_worth_building(of, A);
            *of_resident = copies.given;
            resident = copies.merged;
        } else if (!A->merged) {
            resident = resident_worth_building(A, nullptr).given;
        }
        if (rl.nchunks != 0 && (t_options.spmm_slab == 1 || resident)) {
            try {
                blk_ptr.resize((size_t)lay.P * rl.nblk + 1);
                blk_src.resize((size_t)rl.nchunks * MC_CHUNK);
                blk_ends.resize((size_t)resident_end_words(A));
                blk_recs.resize((size_t)((resident_records(A) + RESIDENT_PADDING) * resident_rec_bytes(A))); // (readers run ahead of the end)
                if (A->uniform_chunks == 0 && rl.nblk > 1) {
                    order.resize((size_t)lay.P);
                    for (int p = 0; p < lay.P; ++p) order[(size_t)p] = p;
                    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return row_ptr[x + 1] - row_ptr[x] > row_ptr[y + 1] - row_ptr[y]; });
                }
                rc = mc_resident_pack(K, V, lhs_bits, lay.P, row_ptr, col_idx, values, rl, blk_ptr.data(), blk_recs.data(), blk_src.data(), blk_ends.data());
                if (A->uniform_chunks == 0 && rl.nblk == 1) {
                    splits.resize(RESIDENT_SPLITS + 1);
                    for (int i = 0, p = 0; i <= RESIDENT_SPLITS; ++i) {
                        const int64_t want = rl.nchunks * i / RESIDENT_SPLITS;
                        while (p < lay.P && (blk_ptr[(size_t)p] < want || (i == RESIDENT_SPLITS))) ++p;
                        splits[(size_t)i] = p;
                    }
                }
            } catch (const std::bad_alloc &) {
                free_device(A);
                delete A;
                return MC_ENOMEM;
            }
            if (rc != MC_OK) {
                free_device(A);
                delete A;
                return rc;
            }
        } else {
            A->nblk = 0; A->blk_chunks = 0;
        }
    }
    // The operand with all its columns, where that form is expected to be the fastest for some width of B.  Beside the other copies, not in
    // their place: calls with options, and calls that this form does not take, run in theirs.  (A thread that pins or forbids
    // the other copies gets those and no others.)
    const bool dense_allowed = dense_mode(t_options) == 1 || (dense_mode(t_options) == 0 && t_options.spmm_slab == 0);
    const bool dense = !of && dense_allowed && dense_possible(M, K, lhs_bits) && lay.nvec > 0 && (dense_mode(t_options) == 1 || dense_worth_building(A));
    hipStream_t s = static_cast<hipStream_t>(stream);
#define MC_TRY(call) (ok = ok && hip_ok((call), #call))
    bool ok = true;
    MC_TRY(hipGetDevice(&A->device));
    // the index array gets one spare chunk so that 16-byte index reads never leave it
    // panel pointers, shares and row pointers in one allocation and one copy
    const size_t at_shares = (2 * (size_t)(lay.P + 1) + 3) / 4 * 4, at_rows = at_shares + shares.size();
    try {
        panel_ptr.resize(at_rows + (size_t)lay.P + 1);
    } catch (const std::bad_alloc &) {
        free_device(A);
        delete A;
        return MC_ENOMEM;
    }
    std::copy(shares.begin(), shares.end(), panel_ptr.begin() + at_shares);
    std::copy(row_ptr, row_ptr + lay.P + 1, panel_ptr.begin() + at_rows);
    MC_TRY(hipMalloc(&A->d_panel_ptr, sizeof(int32_t) * panel_ptr.size()));
    A->d_shares = A->d_panel_ptr + at_shares; A->d_row_ptr = A->d_panel_ptr + at_rows;
    MC_TRY(hipMalloc(&A->d_slot_idx, sizeof(int32_t) * (size_t)(lay.nslots + MC_CHUNK)));
    if (lay.vals_bytes) MC_TRY(hipMalloc(&A->d_vals, (size_t)lay.vals_bytes));
    MC_TRY(hipMemcpyAsync(A->d_panel_ptr, panel_ptr.data(), sizeof(int32_t) * panel_ptr.size(), hipMemcpyHostToDevice, s));
    if (lay.nslots)
        MC_TRY(hipMemcpyAsync(A->d_slot_idx, slot_idx.data(), sizeof(int32_t) * (size_t)lay.nslots, hipMemcpyHostToDevice, s));
    if (lay.vals_bytes)
        MC_TRY(hipMemcpyAsync(A->d_vals, vals.data(), (size_t)lay.vals_bytes, hipMemcpyHostToDevice, s));
    std::vector<int32_t> chunk_vec;
    if (lhs_bits != 0 && lay.nslots) {
        try {
            chunk_vec.resize(2 * (size_t)(lay.nslots / MC_CHUNK));
        } catch (const std::bad_alloc &) {
            free_device(A);
            delete A;
            return MC_ENOMEM;
        }
        for (int p = 0; p < lay.P; ++p)
            for (int v = row_ptr[p], c = panel_ptr[2 * (size_t)p] / MC_CHUNK; v < row_ptr[p + 1]; v += MC_CHUNK, ++c) {
                chunk_vec[2 * (size_t)c] = v;
                chunk_vec[2 * (size_t)c + 1] = std::min(MC_CHUNK, row_ptr[p + 1] - v);
            }
        MC_TRY(hipMalloc(&A->d_chunk_vec, sizeof(int32_t) * chunk_vec.size()));
        MC_TRY(hipMemcpyAsync(A->d_chunk_vec, chunk_vec.data(), sizeof(int32_t) * chunk_vec.size(), hipMemcpyHostToDevice, s));
    }
    if (A->n_items) {
        MC_TRY(hipMalloc(&A->d_items, sizeof(int32_t) * items.size()));
        MC_TRY(hipMalloc(&A->d_split_panels, sizeof(int32_t) * split_panels.size()));
        MC_TRY(hipMemcpyAsync(A->d_items, items.data(), sizeof(int32_t) * items.size(), hipMemcpyHostToDevice, s));
        MC_TRY(hipMemcpyAsync(A->d_split_panels, split_panels.data(), sizeof(int32_t) * split_panels.size(),
                              hipMemcpyHostToDevice, s));
    }
    if (A->blk_chunks) {
        MC_TRY(hipMalloc(&A->d_blk_ptr, sizeof(int32_t) * blk_ptr.size()));
        MC_TRY(hipMalloc(&A->d_blk_recs, blk_recs.size()));
        MC_TRY(hipMalloc(&A->d_blk_ends, sizeof(uint32_t) * blk_ends.size()));
        MC_TRY(hipMemcpyAsync(A->d_blk_ends, blk_ends.data(), sizeof(uint32_t) * blk_ends.size(), hipMemcpyHostToDevice, s));
        MC_TRY(hipMalloc(&A->d_blk_src, sizeof(int32_t) * blk_src.size()));
        MC_TRY(hipMemcpyAsync(A->d_blk_ptr, blk_ptr.data(), sizeof(int32_t) * blk_ptr.size(), hipMemcpyHostToDevice, s));
        MC_TRY(hipMemcpyAsync(A->d_blk_recs, blk_recs.data(), blk_recs.size(), hipMemcpyHostToDevice, s));
        MC_TRY(hipMemcpyAsync(A->d_blk_src, blk_src.data(), sizeof(int32_t) * blk_src.size(), hipMemcpyHostToDevice, s));
        if (!order.empty()) {
            MC_TRY(hipMalloc(&A->d_order, sizeof(int32_t) * order.size()));
            MC_TRY(hipMemcpyAsync(A->d_order, order.data(), sizeof(int32_t) * order.size(), hipMemcpyHostToDevice, s));
        }
        if (!splits.empty()) {
            MC_TRY(hipMalloc(&A->d_splits, sizeof(int32_t) * splits.size()));
            MC_TRY(hipMemcpyAsync(A->d_splits, splits.data(), sizeof(int32_t) * splits.size(), hipMemcpyHostToDevice, s));
        }
        A->blk_valid = true;
    }
    if (!class_panels.empty()) {
        MC_TRY(hipMalloc(&A->d_class_panels, sizeof(int32_t) * class_panels.size()));
        MC_TRY(hipMemcpyAsync(A->d_class_panels, class_panels.data(), sizeof(int32_t) * class_panels.size(), hipMemcpyHostToDevice, s));
    }
    if (A->merged) {
        MC_TRY(hipMalloc(&A->d_merge_src, sizeof(int32_t) * m_src.size()));
        MC_TRY(hipMemcpyAsync(A->d_merge_src, m_src.data(), sizeof(int32_t) * m_src.size(), hipMemcpyHostToDevice, s));
        A->merged_valid = true;
    }
    // (last, and left out where there is no memory for it: no call depends on it)
    if (ok && dense) {
        if (hipMalloc(&A->d_dense, (size_t)dense_bytes(M, K, lhs_bits)) == hipSuccess) {
            MC_TRY(launch_dense_fill(dense_fill_args(A), s));
            A->dense_valid = true;
        } else {
            A->d_dense = nullptr;
            (void)hipGetLastError();
        }
    }
    MC_TRY(hipStreamSynchronize(s)); // host staging buffers die at return
#undef MC_TRY
    if (!ok) {
        free_device(A);
        delete A;
        return MC_EHIP;
    }
    *out = A;
    return MC_OK;
}
} // namespace

extern "C" int mc_mat_create(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx,
                             const void *values, void *stream, mc_mat **out)
{
    return mat_create_impl(M, K, V, lhs_bits, row_ptr, col_idx, values, stream, nullptr, nullptr, out);
}

extern "C" int mc_mat_merged_info(const mc_mat *A, int *group, int64_t *nvec)
{
    if (!A) return MC_EINVAL;
    if (group) *group = A->merged ? A->merge_group : 0;
    if (nvec) *nvec = A->merged ? A->merged->nvec : 0;
    return MC_OK;
}

extern "C" void mc_mat_destroy(mc_mat *A)
{
    if (!A) return;
    free_device(A);
    delete A;
}

extern "C" int mc_mat_info(const mc_mat *A, int *M, int *K, int *V, int *lhs_bits, int64_t *nvec, int64_t *nslots)
{
    if (!A) return MC_EINVAL;
    if (M) *M = A->M;
    if (K) *K = A->K;
    if (V) *V = A->V;
    if (lhs_bits) *lhs_bits = A->lhs_bits;
    if (nvec) *nvec = A->nvec;
    if (nslots) *nslots = A->nslots;
    return MC_OK;
}

extern "C" int mc_mat_set_values_device(mc_mat *A, const void *values_dev, void *stream)
{
    if (!A) return MC_EINVAL;
    if (A->lhs_bits == 0) return MC_EINVAL;        // a pattern-only mask holds no values
    if (A->nslots == 0) return MC_OK;              // no stored vector: nothing to replace
    if (!values_dev) return MC_EINVAL;
    if (!on_device_of(A)) return MC_EINVAL;
    ValuesArgs a = {};
    a.src = static_cast<const uint8_t *>(values_dev);
    a.V = A->V; a.bits = (A->lhs_bits == 12) ? 16 : A->lhs_bits;
    for (mc_mat *X : {A, A->merged}) {
        if (!X) continue;
        const int32_t *merge_src = X == A ? nullptr : A->d_merge_src;
        const int chunk_bytes = MC_CHUNK * X->V * a.bits / 8;
        ValuesJob &panels = a.job[a.njobs++];
        panels = {X->d_chunk_vec, nullptr, merge_src, static_cast<uint8_t *>(X->d_vals), X->nslots / MC_CHUNK, chunk_bytes, 0, X->V, 0, 1};
        if (X->d_blk_recs) { // the LDS-ordered copy follows
            ValuesJob &copy = a.job[a.njobs++];
            copy = {nullptr, X->d_blk_src, merge_src, X->d_blk_recs, X->blk_chunks, resident_rec_bytes(X), rec_chunks(X) * 2 * MC_CHUNK, X->V, 0, rec_chunks(X)};
        }
    }
    MC_HIP(launch_set_values(a, static_cast<hipStream_t>(stream)));
    // (The copy with all columns takes longer to write than one product gains by it, 13 us against 7 at 4096 x 4096, V = 2, half empty, N = 512: where it
    // was neither asked for nor read, products go back to the other forms.  One that read it may be part of a graph and read it again.)
    A->dense_valid = false;
    if (A->d_dense && (A->dense_asked || A->dense_read.load(std::memory_order_relaxed))) {
        MC_HIP(launch_dense_fill(dense_fill_args(A), static_cast<hipStream_t>(stream)));
        A->dense_valid = true;
    }
    A->blk_valid = A->d_blk_recs != nullptr;
    if (A->merged) {
        A->merged->blk_valid = A->merged->d_blk_recs != nullptr;
        A->merged_valid = true;
    }
    return MC_OK;
}

namespace {
// The form one SpMM call takes: the operand or its merged copy, and whether rows of B are resident in LDS (then plan is
// the work split), or the operand with all its columns (dense: the tile shape, else -1), or else gathered as planned.
struct SpmmForm { const mc_mat *A; bool slab; SlabPlan plan; int dense; GatherPlan gather; };

// ldb_bytes: from row to row of B; out_mode as in spmm_impl
SpmmForm spmm_form(const mc_mat *A, int row_bytes, int64_t ldb_bytes, int rb, int out_mode, unsigned flags, const mc_options &o)
{
    const bool r4 = rb == 4;
    const int out_bytes = out_mode == 2 ? 2 : 4;
    const bool slab_possible = o.spmm_slab != -1 && flags == 0 && rb != 16 && o.spmm_row_tile_bytes == 0 && o.spmm_waves == 0;
    // a 16-row panel leaves no MFMA row for the column sums that unsigned operands need
    const bool merged_possible = A->merged && A->merged_valid && o.spmm_merge != -1 && !(flags != 0 && A->merged->V > 8);
    SpmmForm f = {A, false, {}, -1, {0, 0, 1e30}};
    f.plan.us = 1e30;
    const mc_mat *resident_on = A;
    for (int m = (merged_possible && o.spmm_merge == 1) ? 1 : 0; m <= (merged_possible ? 1 : 0); ++m) {
        const mc_mat *X = m ? A->merged : A;
        const bool slab = slab_possible && X->d_blk_recs && X->blk_valid;
        SlabPlan pl;
        pl.us = 1e30;
        if (slab) plan_slab(X, row_bytes, r4, out_bytes, o, &pl);
        if (pl.us < f.plan.us) { f.plan = pl; resident_on = X; }
        if (!slab || o.spmm_slab != 1) {
            const GatherPlan gather = plan_gather(X, X->lhs_bits, row_bytes, rb, out_bytes, 1, takes_items(X, out_mode, o),
                                                  spmm_stages_for(o, X->K, ldb_bytes, row_bytes), flags != 0, o);
            if (gather.us < f.gather.us) { f.gather = gather; f.A = X; }
        }
    }
    // (The resident form with 3 % on: the fit is for operands in turn; where one comes again and again its A and indices are in L2 and a gather
    // takes up to 17 % less.  On the 168 points of bench.py --sweep the form and variant picked are 2.3 % over the fastest in turn and 3.3 % warm, without
    // the 3 % 2.45 and 3.7 %; on 2280 drawn operands in turn 2.87 and 2.78 %.)
    f.slab = 1.03 * f.plan.us < f.gather.us;
    if (f.slab) f.A = resident_on;
    const bool dense_wanted = dense_mode(o) == 1 || (dense_mode(o) == 0 && !pins_other_form(o));
    if (A->d_dense && A->dense_valid && dense_wanted && flags == 0 && rb != 16 && o.spmm_slab == 0 &&
        o.spmm_row_tile_bytes == 0 && o.spmm_waves == 0 && (A->K - 1) * ldb_bytes + row_bytes <= INT32_MAX && (A->K + 8192) * ldb_bytes <= UINT32_MAX) {
        const DensePlan d = plan_dense(A->M, A->K, A->lhs_bits, row_bytes, r4, out_bytes, dense_tile(o));
        // (its expected times and the others' were fitted apart, and where several of theirs compete the least is too low: with 3 % off the form and
        // variant picked for 1437 drawn operands are 2.88 % slower than the fastest on average, with nothing 2.95 %, with 3 % on 3.0 %)
        if (d.tile >= 0 && (dense_mode(o) == 1 || 0.97 * d.us < (f.slab ? f.plan.us : f.gather.us))) {
            f.A = A; f.slab = false; f.dense = d.tile; f.plan.us = d.us;
        }
    }
    return f;
}

// out_mode 0: int32 results; 1 / 2: scale * result as fp32 / fp16 (fused dequantisation)
int spmm_impl(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, unsigned flags, int out_mode,
              float scale, void *C_dev, int ldc, const mc_options *opts, void *stream)
{
    if (!A || !B_dev || !C_dev) return MC_EINVAL;
    mc_options o;
    if (resolve_options(opts, &o) != MC_OK) return MC_EINVAL;
    if (!valid_prec((int)prec)) return MC_EUNSUPPORTED;
    if (flags & ~(unsigned)(MC_LHS_UNSIGNED | MC_RHS_UNSIGNED)) return MC_EINVAL;
    if (flags && prec != MC_L8R8 && prec != MC_L8R4 && prec != MC_L4R4) return MC_EUNSUPPORTED;
    // (a matrix without any stored vector has no value buffer and is a valid all-zero operand)
    if ((!A->d_vals && A->nslots > 0) || A->lhs_bits != lhs_bits_of(prec)) return MC_EINVAL;
    const int rb = rhs_bits_of(prec);
    if (N <= 0 || N % (128 / rb) != 0) return MC_EINVAL; // whole 16-byte pieces of a row
    if (ldb < N || ldc < N) return MC_EINVAL;
    if (((int64_t)ldb * rb / 8) % 16 != 0 || ldc % 4 != 0) return MC_EALIGN;
    if (!aligned16(B_dev) || !aligned16(C_dev)) return MC_EALIGN;
    if (rb == 4 && A->K > ((flags != 0) ? 32768 : 131072)) return MC_EUNSUPPORTED;
    if (out_mode && !std::isfinite(scale)) return MC_EINVAL;
    if (!on_device_of(A)) return MC_EINVAL;

    // the operand's merged copy (panels of 8 or 16 rows at the union of their columns) where it is expected to be faster
    const int rows = A->M;
    const SpmmForm form = spmm_form(A, N * rb / 8, (int64_t)ldb * rb / 8, rb, out_mode, flags, o);
    A = form.A;

    SpmmArgs a = {};
    a.rows = rows;
    a.lhs_unsigned = (flags & MC_LHS_UNSIGNED) ? 1 : 0; a.rhs_unsigned = (flags & MC_RHS_UNSIGNED) ? 1 : 0;
    a.panel_ptr = A->d_panel_ptr; a.slot_idx = A->d_slot_idx;
    a.vals = A->d_vals; a.vals_batch_stride = 0;
    a.B = static_cast<const uint8_t *>(B_dev); a.ldb_bytes = (int64_t)ldb * rb / 8; a.B_batch_stride = 0;
    a.row_bytes = N * rb / 8;
    a.C = C_dev; a.ldc = ldc; a.C_batch_stride = 0;
    a.P = A->P; a.V = A->V; a.batch = 1; a.float_out = out_mode; a.out_scale = out_mode ? scale : 1.f;
    if (form.dense >= 0) {
        A->dense_read.store(true, std::memory_order_relaxed);
        DenseArgs da = {};
        da.A = A->d_dense; da.a_bytes = (int)dense_bytes(A->M, A->K, A->lhs_bits);
        da.nrb = (A->M + 15) / 16; da.nch = (A->K + MC_CHUNK - 1) / MC_CHUNK;
        da.B = a.B; da.ldb_bytes = a.ldb_bytes; da.b_bytes = (int)((A->K - 1) * a.ldb_bytes + a.row_bytes); da.cols = N;
        da.C = C_dev; da.ldc = ldc; da.rows = rows; da.float_out = out_mode; da.out_scale = a.out_scale;
        MC_HIP(launch_spmm_dense(prec, da, form.dense, static_cast<hipStream_t>(stream)));
        return MC_OK;
    }
    if (form.slab) {
        const SlabPlan &pl = form.plan;
        SlabArgs sa = {};
        sa.blk_ptr = A->d_blk_ptr; sa.recs = A->d_blk_recs; sa.ends = A->d_blk_ends; sa.end_words = resident_end_words(A);
        sa.order = A->d_order; sa.splits = A->d_splits;
        sa.uniform_chunks = A->uniform_chunks; sa.rec_bytes = resident_rec_bytes(A); sa.nrecs = resident_records(A);
        sa.B = a.B; sa.ldb_bytes = a.ldb_bytes; sa.row_bytes = a.row_bytes; sa.K = A->K;
        sa.C = C_dev; sa.ldc = ldc;
        sa.P = A->P; sa.V = A->V; sa.nblk = A->nblk; sa.block_rows = A->block_rows; sa.nt = A->blk_nt; sa.rows = rows;
        sa.float_out = out_mode; sa.out_scale = a.out_scale;
        sa.ntiles = pl.ntiles; sa.groups = pl.groups; sa.wpp = pl.wpp; sa.waves = pl.waves;
        MC_HIP(launch_spmm_slab(prec, sa, pl.nt, static_cast<hipStream_t>(stream)));
        return MC_OK;
    }
    a.stages = spmm_stages_for(o, A->K, a.ldb_bytes, a.row_bytes);
    a.short_b = spmm_short_b(A->K, a.ldb_bytes, a.row_bytes);
    a.uniform_chunks = A->uniform_chunks;
    a.max_unit_chunks = A->max_panel_chunks;
    if (takes_items(A, out_mode, o)) {
        a.max_unit_chunks = A->max_item_chunks;
        // very unequal panels: long ones are shared by several workgroups that add into cleared rows
        // (integer results only: a scaled, rounded result cannot be accumulated piecewise)
        a.items = A->d_items; a.n_units = A->n_items;
        MC_HIP(launch_zero_rows(static_cast<int32_t *>(C_dev), ldc, N, A->V, A->d_split_panels, A->n_split,
                                static_cast<hipStream_t>(stream)));
    }
    MC_HIP(launch_spmm(prec, a, form.gather.bnb, form.gather.waves, static_cast<hipStream_t>(stream)));
    return MC_OK;
}
} // namespace

extern "C" int mc_spmm(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, int32_t *C_dev, int ldc,
                       void *stream)
{
    return spmm_impl(A, B_dev, N, ldb, prec, 0u, 0, 1.f, C_dev, ldc, nullptr, stream);
}

extern "C" int mc_spmm_flags(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, unsigned flags,
                             int32_t *C_dev, int ldc, void *stream)
{
    return spmm_impl(A, B_dev, N, ldb, prec, flags, 0, 1.f, C_dev, ldc, nullptr, stream);
}

extern "C" int mc_spmm_ex(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, unsigned flags,
                          const mc_options *options, int32_t *C_dev, int ldc, void *stream)
{
    const mc_options automatic = {};
    return spmm_impl(A, B_dev, N, ldb, prec, flags, 0, 1.f, C_dev, ldc, options ? options : &automatic, stream);
}

namespace {
// The options that mc_spmm_form is asked about: the caller's, else automatic ones as in mc_spmm_ex, but for a choice of the copy with all
// columns that the thread has made (mc_set_spmm_dense).
int form_options(const mc_options *given, mc_options *out)
{
    if (given) return resolve_options(given, out);
    *out = mc_options{};
    if (std::abs(t_options.spmm_merge) >= MC_SPMM_DENSE) out->spmm_merge = t_options.spmm_merge;
    return MC_OK;
}
} // namespace

extern "C" int mc_spmm_form(const mc_mat *A, int N, mc_prec prec, const mc_options *options)
{
    if (!A || N <= 0 || !valid_prec((int)prec) || A->lhs_bits != lhs_bits_of(prec)) return MC_EINVAL;
    mc_options o;
    if (form_options(options, &o) != MC_OK) return MC_EINVAL;
    const int rb = rhs_bits_of(prec);
    const SpmmForm form = spmm_form(A, N * rb / 8, (int64_t)N * rb / 8, rb, 0, 0u, o);
    return form.dense >= 0 ? 4 | (A->merged ? 2 : 0) : (form.slab ? 1 : 0) | (form.A != A ? 2 : 0);
}

extern "C" double mc_spmm_form_us(const mc_mat *A, int N, mc_prec prec, int out_bytes, const mc_options *options)
{
    if (!A || N <= 0 || !valid_prec((int)prec) || A->lhs_bits != lhs_bits_of(prec) || (out_bytes != 2 && out_bytes != 4)) return MC_EINVAL;
    mc_options o;
    if (form_options(options, &o) != MC_OK) return MC_EINVAL;
    const int rb = rhs_bits_of(prec);
    const SpmmForm form = spmm_form(A, N * rb / 8, (int64_t)N * rb / 8, rb, out_bytes == 2 ? 2 : 0, 0u, o);
    return form.slab || form.dense >= 0 ? form.plan.us : form.gather.us;
}

extern "C" int mc_spmm_dequant(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, unsigned flags,
                               float scale, mc_out_type out_type, void *C_dev, int ldc, void *stream)
{
    if (out_type != MC_OUT_F32 && out_type != MC_OUT_F16) return MC_EUNSUPPORTED;
    return spmm_impl(A, B_dev, N, ldb, prec, flags, out_type == MC_OUT_F16 ? 2 : 1, scale, C_dev, ldc, nullptr, stream);
}

extern "C" int64_t mc_probe_gather_sink_len(const mc_mat *A, int N, mc_prec prec)
{
    if (!A || N <= 0 || !valid_prec((int)prec)) return 0;
    // the widest tiling (64-byte tiles) bounds the number of workgroups
    return (int64_t)A->P * (((int64_t)N * rhs_bits_of(prec) / 8 + 63) / 64);
}

extern "C" int mc_probe_gather(const mc_mat *A, const void *B_dev, int N, int ldb, mc_prec prec, int32_t *sink_dev,
                               void *stream)
{
    if (!A || !B_dev || !sink_dev) return MC_EINVAL;
    if (!valid_prec((int)prec)) return MC_EUNSUPPORTED;
    const int rb = rhs_bits_of(prec);
    if (N <= 0 || N % (128 / rb) != 0 || ldb < N) return MC_EINVAL;
    if (((int64_t)ldb * rb / 8) % 16 != 0 || !aligned16(B_dev)) return MC_EALIGN;
    if (!on_device_of(A)) return MC_EINVAL;
    const mc_options o = t_options;
    SpmmArgs a = {};
    a.panel_ptr = A->d_panel_ptr; a.slot_idx = A->d_slot_idx;
    a.vals = nullptr; a.vals_batch_stride = 0;
    a.B = static_cast<const uint8_t *>(B_dev); a.ldb_bytes = (int64_t)ldb * rb / 8; a.B_batch_stride = 0;
    a.row_bytes = N * rb / 8;
    a.C = nullptr; a.ldc = 0; a.C_batch_stride = 0;
    a.P = A->P; a.V = A->V; a.rows = A->M; a.batch = 1; a.float_out = 0; a.out_scale = 1.f;
    a.uniform_chunks = A->uniform_chunks;
    const GatherPlan plan = plan_gather(A, A->lhs_bits, a.row_bytes, rb, 4, 1, false, spmm_stages_for(o, A->K, a.ldb_bytes, a.row_bytes), false, o);
    MC_HIP(launch_gather_probe(a, plan.bnb, plan.waves, sink_dev, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int64_t mc_probe_spmm_phases_len(const mc_mat *A, int N)
{
    if (!A || N <= 0) return 0;
    return (int64_t)A->P * ((N + 127) / 128) * 2 * 10;
}

extern "C" int mc_probe_spmm_phases(const mc_mat *A, const void *B_dev, int N, int ldb, int32_t *C_dev, int ldc, int64_t *trace_dev,
                                    void *stream)
{
    if (!A || !B_dev || !C_dev || !trace_dev) return MC_EINVAL;
    if (N <= 0 || N % 16 != 0 || ldb < N || ldc < N) return MC_EINVAL;
    if (ldb % 16 != 0 || ldc % 4 != 0 || !aligned16(B_dev) || !aligned16(C_dev)) return MC_EALIGN;
    if (!on_device_of(A)) return MC_EINVAL;
    const mc_options automatic = {};
    if (A->lhs_bits != 8 || !A->d_vals || A->max_panel_chunks > 2 * 4 || spmm_stages_for(automatic, A->K, ldb, N) != 2)
        return MC_EUNSUPPORTED;
    SpmmArgs a = {};
    a.panel_ptr = A->d_panel_ptr; a.slot_idx = A->d_slot_idx; a.vals = A->d_vals;
    a.B = static_cast<const uint8_t *>(B_dev); a.ldb_bytes = ldb; a.row_bytes = N;
    a.C = C_dev; a.ldc = ldc;
    a.P = A->P; a.V = A->V; a.rows = A->M; a.batch = 1; a.out_scale = 1.f;
    a.stages = 2; a.short_b = 1; a.max_unit_chunks = A->max_panel_chunks; a.uniform_chunks = A->uniform_chunks;
    a.trace = reinterpret_cast<long long *>(trace_dev);
    MC_HIP(launch_spmm_phase_probe(a, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_probe_mfma(int workgroups, int iters, int32_t *sink_dev, void *stream)
{
    if (!sink_dev || workgroups <= 0 || workgroups > 65535 || iters <= 0) return MC_EINVAL;
    MC_HIP(launch_mfma_probe(workgroups, iters, sink_dev, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

namespace {
int sddmm_impl(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, const mc_mat *mask, mc_prec prec,
               unsigned flags, int out_mode, float scale, void *S_dev, const mc_options *opts, void *stream)
{
    if (!Q_dev || !Kmat_dev || !mask) return MC_EINVAL;
    mc_options o;
    if (resolve_options(opts, &o) != MC_OK) return MC_EINVAL;
    if (!S_dev && mask->nvec > 0) return MC_EINVAL; // (a mask without any vector has an empty output)
    if (!valid_prec((int)prec)) return MC_EUNSUPPORTED;
    if (flags & ~(unsigned)(MC_LHS_UNSIGNED | MC_RHS_UNSIGNED)) return MC_EINVAL;
    if (flags && prec != MC_L8R8 && prec != MC_L4R4) return MC_EUNSUPPORTED;
    if (flags && prec == MC_L4R4 && Kd > 32768) return MC_EUNSUPPORTED; // 256x scaled sums stay inside int32
    if (prec != MC_L8R8 && prec != MC_L4R4 && prec != MC_L16R16) return MC_EUNSUPPORTED;
    const int bits = lhs_bits_of(prec);
    if (Kd <= 0 || Kd % (128 / bits) != 0 || ldq < Kd || ldk < Kd) return MC_EINVAL;
    if (((int64_t)ldq * bits / 8) % 16 != 0 || ((int64_t)ldk * bits / 8) % 16 != 0) return MC_EALIGN;
    if (!aligned16(Q_dev) || !aligned16(Kmat_dev) || !aligned16(S_dev)) return MC_EALIGN;
    if (out_mode && !std::isfinite(scale)) return MC_EINVAL;
    if (mask->nvec == 0) return MC_OK;
    if (!on_device_of(mask)) return MC_EINVAL;

    SddmmArgs a = {};
    a.float_out = out_mode; a.out_scale = out_mode ? scale : 1.f;
    a.slot_idx = mask->d_slot_idx;
    a.Q = static_cast<const uint8_t *>(Q_dev); a.ldq_bytes = (int64_t)ldq * bits / 8; a.Q_batch_stride = 0;
    a.Kmat = static_cast<const uint8_t *>(Kmat_dev); a.ldk_bytes = (int64_t)ldk * bits / 8; a.K_batch_stride = 0;
    a.row_bytes = Kd * bits / 8;
    a.S = S_dev; a.S_batch_stride = 0;
    a.V = mask->V; a.batch = 1;
    a.lhs_unsigned = (flags & MC_LHS_UNSIGNED) ? 1 : 0; a.rhs_unsigned = (flags & MC_RHS_UNSIGNED) ? 1 : 0;
    take_shares(mask, o.spmm_splitting != -1, &a);
    MC_HIP(launch_sddmm(bits, a, choose_sddmm_waves(mask, a.n_shares, 1, a.row_bytes, bits, o), static_cast<hipStream_t>(stream)));
    return MC_OK;
}
} // namespace

extern "C" int mc_sddmm(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, const mc_mat *mask,
                        mc_prec prec, int32_t *S_dev, void *stream)
{
    return sddmm_impl(Q_dev, ldq, Kmat_dev, ldk, Kd, mask, prec, 0u, 0, 1.f, S_dev, nullptr, stream);
}

extern "C" int mc_sddmm_flags(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, const mc_mat *mask,
                              mc_prec prec, unsigned flags, int32_t *S_dev, void *stream)
{
    return sddmm_impl(Q_dev, ldq, Kmat_dev, ldk, Kd, mask, prec, flags, 0, 1.f, S_dev, nullptr, stream);
}

extern "C" int mc_sddmm_ex(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, const mc_mat *mask,
                           mc_prec prec, unsigned flags, const mc_options *options, int32_t *S_dev, void *stream)
{
    const mc_options automatic = {};
    return sddmm_impl(Q_dev, ldq, Kmat_dev, ldk, Kd, mask, prec, flags, 0, 1.f, S_dev, options ? options : &automatic, stream);
}

extern "C" int mc_sddmm_dequant(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, const mc_mat *mask,
                                mc_prec prec, unsigned flags, float scale, mc_out_type out_type, void *S_dev,
                                void *stream)
{
    if (out_type != MC_OUT_F32 && out_type != MC_OUT_F16) return MC_EUNSUPPORTED;
    return sddmm_impl(Q_dev, ldq, Kmat_dev, ldk, Kd, mask, prec, flags, out_type == MC_OUT_F16 ? 2 : 1, scale, S_dev,
                      nullptr, stream);
}

extern "C" int mc_sddmm_to_mat(const void *Q_dev, int ldq, const void *Kmat_dev, int ldk, int Kd, mc_prec prec, float scale,
                               mc_mat *P, void *stream)
{
    if (!Q_dev || !Kmat_dev || !P) return MC_EINVAL;
    if (prec != MC_L8R8 && prec != MC_L4R4 && prec != MC_L16R16) return MC_EUNSUPPORTED;
    if (P->lhs_bits == 0) return MC_EINVAL;                      // a pattern-only mask has no values to receive the codes
    if (P->lhs_bits != 8 && P->lhs_bits != 16) return MC_EUNSUPPORTED;
    const int bits = lhs_bits_of(prec);
    if (Kd <= 0 || Kd % (128 / bits) != 0 || ldq < Kd || ldk < Kd) return MC_EINVAL;
    if (((int64_t)ldq * bits / 8) % 16 != 0 || ((int64_t)ldk * bits / 8) % 16 != 0) return MC_EALIGN;
    if (!aligned16(Q_dev) || !aligned16(Kmat_dev)) return MC_EALIGN;
    if (!std::isfinite(scale)) return MC_EINVAL;
    if (P->nvec == 0) return MC_OK;
    if (!on_device_of(P)) return MC_EINVAL;
    const mc_options o = t_options;

    SddmmArgs a = {};
    a.float_out = 3; a.out_scale = scale;
    a.dev_vals = P->d_vals; a.dev_batch_stride = 0; a.code_bits = P->lhs_bits;
    a.slot_idx = P->d_slot_idx;
    a.Q = static_cast<const uint8_t *>(Q_dev); a.ldq_bytes = (int64_t)ldq * bits / 8; a.Q_batch_stride = 0;
    a.Kmat = static_cast<const uint8_t *>(Kmat_dev); a.ldk_bytes = (int64_t)ldk * bits / 8; a.K_batch_stride = 0;
    a.row_bytes = Kd * bits / 8;
    a.S = nullptr; a.S_batch_stride = 0;
    a.V = P->V; a.batch = 1;
    take_shares(P, o.spmm_splitting != -1, &a);
    P->blk_valid = false; // only the panel format receives the new values
    P->merged_valid = false;
    P->dense_valid = false;
    MC_HIP(launch_sddmm(bits, a, choose_sddmm_waves(P, a.n_shares, 1, a.row_bytes, bits, o), static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_absmax(const float *x_dev, int64_t n, float *result_dev, void *stream)
{
    if (!x_dev || !result_dev || n < 0) return MC_EINVAL;
    if (!aligned16(x_dev)) return MC_EALIGN;
    MC_HIP(launch_absmax(x_dev, n, result_dev, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_quantize(const float *x_dev, int64_t n, float scale, int bits, void *q_dev, void *stream)
{
    if (!x_dev || !q_dev || n < 0) return MC_EINVAL;
    if (bits != 8 && bits != 4) return MC_EUNSUPPORTED;
    if (!(scale > 0.f) || !std::isfinite(scale) || (bits == 4 && n % 2 != 0)) return MC_EINVAL;
    if (!aligned16(x_dev) || (reinterpret_cast<uintptr_t>(q_dev) & 7u) != 0) return MC_EALIGN;
    MC_HIP(launch_quantize(x_dev, n, scale, bits, static_cast<uint8_t *>(q_dev), static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_sparse_softmax_bits(const mc_mat *mask, int batch, const int32_t *S_dev, float score_scale,
                                      float inv_s_p, int code_bits, void *codes_dev, void *stream)
{
    if (!mask || batch <= 0) return MC_EINVAL;
    if ((!S_dev || !codes_dev) && mask->nvec > 0) return MC_EINVAL;
    if (code_bits != 8 && code_bits != 16) return MC_EUNSUPPORTED;
    if (!std::isfinite(score_scale) || !std::isfinite(inv_s_p)) return MC_EINVAL;
    if (mask->nvec == 0) return MC_OK; // nothing stored: empty input and output
    if (!on_device_of(mask)) return MC_EINVAL;
    const mc_options o = t_options;
    SoftmaxArgs a = {};
    a.row_ptr = mask->d_row_ptr; a.S = S_dev; a.codes = codes_dev;
    a.batch_stride = mask->nvec * mask->V;
    a.score_scale = score_scale; a.inv_s_p = inv_s_p;
    a.P = mask->P; a.V = mask->V; a.batch = batch; a.code_bits = code_bits;
    a.max_panel_chunks = mask->max_panel_chunks; a.variant = o.softmax_variant;
    MC_HIP(launch_softmax(a, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_sparse_softmax_to_mat(mc_mat *P, const int32_t *S_dev, float score_scale, float inv_s_p, void *stream)
{
    if (!P || !S_dev) return MC_EINVAL;
    if (P->lhs_bits == 0) return MC_EINVAL;
    if (P->nslots == 0) return MC_OK;
    if (P->lhs_bits != 8 && P->lhs_bits != 16) return MC_EUNSUPPORTED;
    if (!std::isfinite(score_scale) || !std::isfinite(inv_s_p)) return MC_EINVAL;
    if (!on_device_of(P)) return MC_EINVAL;
    const mc_options o = t_options;
    SoftmaxArgs a = {};
    a.row_ptr = P->d_row_ptr; a.S = S_dev; a.codes = nullptr;
    a.panel_ptr = P->d_panel_ptr; a.dev_vals = P->d_vals; a.dev_batch_stride = 0;
    a.batch_stride = P->nvec * P->V;
    a.score_scale = score_scale; a.inv_s_p = inv_s_p;
    a.P = P->P; a.V = P->V; a.batch = 1; a.code_bits = P->lhs_bits;
    a.max_panel_chunks = P->max_panel_chunks; a.variant = o.softmax_variant;
    P->blk_valid = false; // only the panel format receives the new values
    P->merged_valid = false;
    P->dense_valid = false;
    MC_HIP(launch_softmax(a, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

extern "C" int mc_sparse_softmax(const mc_mat *mask, int batch, const int32_t *S_dev, float score_scale,
                                 float inv_s_p, int8_t *codes_dev, void *stream)
{
    return mc_sparse_softmax_bits(mask, batch, S_dev, score_scale, inv_s_p, 8, codes_dev, stream);
}

namespace {
inline size_t round256(size_t x) { return (x + 255) / 256 * 256; }
struct AttnWs { size_t scores, vals, acc, total; };
// with_scores: the int32 scores of all heads travel through the workspace too (the three-kernel form).
// acc_dk != 0: room for the int32 output rows (acc_dk columns) of the panels that several workgroups share.
AttnWs attn_layout(int heads, const mc_mat *mask, int p_bits, bool with_scores = true, int acc_dk = 0)
{
    AttnWs w;
    const size_t nnz = (size_t)mask->nvec * mask->V, pb = (size_t)p_bits / 8;
    w.scores = 0;
    w.vals = w.scores + (with_scores ? round256((size_t)heads * nnz * sizeof(int32_t)) : 0);
    w.acc = w.vals + round256((size_t)heads * (size_t)mask->nslots * mask->V * pb);
    w.total = w.acc + round256((size_t)heads * (size_t)mask->n_split * mask->V * (size_t)acc_dk * sizeof(int32_t));
    return w;
}
// Whether the pipeline's SpMM shares long panels between workgroups (it then needs the extra workspace rows).
// Only on request: on masks whose panel lengths are log-normal (sigma 0.5 .. 1.5, 4096 x 4096, 1 .. 8 heads) it was
// 1 - 10 % slower than whole panels, the pieces of a mask being short (made for the SDDMM, which needs no atomics)
// and the layer's time being that of the scores of the long panels anyway.
inline bool pipeline_splits(const mc_mat *mask, const mc_options &o) { return mask->n_items > 0 && o.spmm_splitting == 1; }

// Waves per (panel, head) of the kernel that computes scores and softmax together, or 0 when the layer has to
// run as three kernels (rows longer than 256 bytes, a panel whose scores do not fit LDS, or pinned by the options).
int scores_kernel_waves(const mc_mat *mask, int heads, int dk, int qkv_bits, const mc_options &o)
{
    const int row_bytes = dk * qkv_bits / 8;
    if (o.attention_mode == 6 || row_bytes > 256) return 0;
    // four waves share a panel's chunks when it has at least three (8 heads x 4096 x 64 at 90 %: 27.2 us with two
    // waves, 21.9 with four), unless the options pin the count
    const double avg = mask->P ? (double)(mask->nslots / MC_CHUNK) / mask->P : 0.0;
    int w = o.sddmm_waves > 0 ? (o.sddmm_waves >= 4 ? 4 : 2) : (avg >= 3.0 ? 4 : 2);
    // long panels: fewer waves leave more LDS for the scores
    while (w > 2 && mask->max_panel_chunks * MC_CHUNK > scores_softmax_max_npad(row_bytes, w)) w /= 2;
    return mask->max_panel_chunks * MC_CHUNK <= scores_softmax_max_npad(row_bytes, w) ? w : 0;
}

// SDDMM -> softmax (writing the SpMM's operand format) -> SpMM, every step a kernel of its own; intermediates in the
// workspace.  Strides of Q/Km/Vm in bytes, of O in elements.
int attention_pipeline(const uint8_t *Q, const uint8_t *Km, const uint8_t *Vm, int heads, int dk, int qkv_bits,
                       int p_bits, int64_t head_stride_bytes, int64_t token_stride_bytes, int64_t o_head_stride,
                       int64_t o_token_stride, const mc_mat *mask, float s_q, float s_k, float s_v, float s_p,
                       void *O, int out_f16, void *workspace_dev, bool split_panels, const mc_options &o, hipStream_t s)
{
    const int sw = scores_kernel_waves(mask, heads, dk, qkv_bits, o);
    const AttnWs ws = attn_layout(heads, mask, p_bits, sw == 0, split_panels ? dk : 0);
    const int64_t nnz = mask->nvec * mask->V;
    uint8_t *wsb = static_cast<uint8_t *>(workspace_dev);
    int32_t *scores = reinterpret_cast<int32_t *>(wsb + ws.scores);
    uint8_t *pvals = wsb + ws.vals;
    const int row_bytes = dk * qkv_bits / 8, pb = p_bits / 8;

    if (sw) {
        // scores and softmax in one kernel: the scores stay in LDS, only the codes (in the layout the SpMM
        // reads: Section 4.3 lets the producer pick the output format by the consumer) reach memory
        ScoresArgs c = {};
        c.panel_ptr = mask->d_panel_ptr; c.slot_idx = mask->d_slot_idx;
        c.Q = Q; c.Km = Km; c.in_head_stride = head_stride_bytes; c.in_token_stride = token_stride_bytes;
        c.row_bytes = row_bytes;
        c.score_scale = s_q * s_k / std::sqrt((float)dk); c.inv_s_p = 1.f / s_p;
        c.dev_vals = pvals; c.dev_batch_stride = mask->nslots * 8 * pb;
        c.P = mask->P; c.heads = heads; c.max_npad = mask->max_panel_chunks * MC_CHUNK;
        MC_HIP(launch_scores_softmax(c, qkv_bits, p_bits, sw, s));
    } else {
        SddmmArgs d = {};
        d.slot_idx = mask->d_slot_idx;
        d.Q = Q; d.ldq_bytes = token_stride_bytes; d.Q_batch_stride = head_stride_bytes;
        d.Kmat = Km; d.ldk_bytes = token_stride_bytes; d.K_batch_stride = head_stride_bytes;
        d.row_bytes = row_bytes; d.S = scores; d.S_batch_stride = nnz;
        d.V = 8; d.batch = heads;
        take_shares(mask, o.spmm_splitting != -1, &d);
        MC_HIP(launch_sddmm(qkv_bits, d, choose_sddmm_waves(mask, d.n_shares, heads, row_bytes, qkv_bits, o), s));

        // the softmax writes its codes in the layout the SpMM reads
        SoftmaxArgs f = {};
        f.row_ptr = mask->d_row_ptr; f.S = scores; f.batch_stride = nnz;
        f.codes = nullptr; f.panel_ptr = mask->d_panel_ptr; f.dev_vals = pvals; f.dev_batch_stride = mask->nslots * 8 * pb;
        f.score_scale = s_q * s_k / std::sqrt((float)dk); f.inv_s_p = 1.f / s_p;
        f.P = mask->P; f.V = 8; f.batch = heads; f.code_bits = p_bits;
        f.max_panel_chunks = mask->max_panel_chunks; f.variant = o.softmax_variant;
        MC_HIP(launch_softmax(f, s));
    }

    SpmmArgs m = {};
    m.panel_ptr = mask->d_panel_ptr; m.slot_idx = mask->d_slot_idx;
    m.vals = pvals; m.vals_batch_stride = mask->nslots * 8 * pb;
    m.B = Vm; m.ldb_bytes = token_stride_bytes; m.B_batch_stride = head_stride_bytes;
    m.row_bytes = row_bytes; m.C = O; m.ldc = o_token_stride; m.C_batch_stride = o_head_stride;
    m.P = mask->P; m.V = 8; m.rows = mask->M; m.batch = heads; m.float_out = out_f16 ? 2 : 1; m.out_scale = s_p * s_v;
    m.stages = spmm_stages_for(o, mask->K, m.ldb_bytes, m.row_bytes);
    m.short_b = spmm_short_b(mask->K, m.ldb_bytes, m.row_bytes);
    m.uniform_chunks = mask->uniform_chunks;
    m.max_unit_chunks = mask->max_panel_chunks;
    if (split_panels) {
        // Very unequal panels: the long ones are shared by several workgroups.  A rounded result cannot be added
        // up piecewise, so those add their exact int32 tiles into rows of the workspace (cleared first), which a
        // last small kernel scales and writes to O; all other panels write O directly, as without the split.
        m.items = mask->d_items; m.n_units = mask->n_items; m.max_unit_chunks = mask->max_item_chunks;
        m.acc = reinterpret_cast<int32_t *>(wsb + ws.acc); m.acc_ld = dk; m.n_split = mask->n_split;
        MC_HIP(launch_zero_ints(m.acc, (int64_t)heads * mask->n_split * 8 * dk, s));
    }
    const GatherPlan plan = plan_gather(mask, p_bits, m.row_bytes, qkv_bits, out_f16 ? 2 : 4, heads, split_panels, m.stages, false, o);
    const mc_prec prec = (p_bits == 16) ? (qkv_bits == 4 ? MC_L16R4 : MC_L16R8) : (qkv_bits == 4 ? MC_L8R4 : MC_L8R8);
    MC_HIP(launch_spmm(prec, m, plan.bnb, plan.waves, s));
    if (split_panels)
        MC_HIP(launch_finish_split_rows(m.acc, dk, mask->n_split, 8, heads, mask->d_split_panels, O, o_token_stride,
                                        o_head_stride, m.float_out, m.out_scale, s));
    return MC_OK;
}

// The head dimension of the fused kernel that takes this layer; 0: the pipeline of separate kernels does.
// (Rows of whole 16-byte pieces; dimensions below 64, between 64 and 128 and above run in the next larger tile with the
// missing pieces read as zeros.  Above 128: panels that four waves can share, and not where the caller pins a mode or asks
// for the pipeline's sharing of long panels.  One launch for all batch items against two for each: batch 8, 8 heads x 616, dk = 160,
// 87 % empty: 98 -> 25 us.)
int fused_tile(const mc_mat *mask, int dk, int qkv_bits, const mc_options &o)
{
    if (o.attention_mode == 1 || o.attention_mode == 6 || (dk * qkv_bits / 8) % 16 != 0) return 0;
    if (dk <= 128) return mask->max_panel_chunks * MC_CHUNK <= attention_fused_max_vectors() ? (dk <= 64 ? 64 : 128) : 0;
    return o.attention_mode == 0 && dk <= 192 && mask->max_panel_chunks <= 32 && !pipeline_splits(mask, o) ? 192 : 0;
}

// Memory the library itself provides to callers that cannot allocate (mc_sparse_attention_static):
// one array per GPU, in that GPU's memory for the life of the process; its address on each device is
// looked up once, with that device current.
constexpr size_t STATIC_SCRATCH_BYTES = MC_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES] = {};
std::mutex g_scratch_mutex;

int static_scratch(void **ptr)
{
    int dev = -1;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return MC_EHIP;
    if (dev < 0 || dev >= MAX_DEVICES) return MC_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)")) return MC_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return MC_OK;
}

// use_static: the intermediates of the kernel pipeline go to the library's per-device array instead
// of a caller's workspace
int attention_impl(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int batch, int heads, int L, int dk,
                   int64_t batch_stride, int64_t head_stride, int64_t token_stride, const mc_mat *mask, int p_bits,
                   int qkv_bits, float s_q, float s_k, float s_v, float s_p, mc_out_type out_type, void *O_dev,
                   void *workspace_dev, size_t workspace_bytes, bool use_static, const mc_options *opts, void *stream)
{
    if (out_type != MC_OUT_F32 && out_type != MC_OUT_F16) return MC_EUNSUPPORTED;
    const int out_f16 = (out_type == MC_OUT_F16) ? 1 : 0;
    if (!Q_dev || !Km_dev || !Vm_dev || !mask || !O_dev) return MC_EINVAL;
    mc_options o;
    if (resolve_options(opts, &o) != MC_OK) return MC_EINVAL;
    if ((p_bits != 8 && p_bits != 16) || (qkv_bits != 8 && qkv_bits != 4)) return MC_EUNSUPPORTED;
    const int epp = 128 / qkv_bits; // elements per 16-byte piece
    if (batch <= 0 || batch > 65535 || heads <= 0 || L <= 0 || dk <= 0 || dk % epp != 0) return MC_EINVAL;
    if (mask->M != L || mask->K != L || mask->V != 8) return MC_EINVAL;
    // symmetric quantisation scales are positive; the fused kernel takes the row maximum on the
    // integer scores, which is the maximum of the scaled ones only for a positive scale
    if (!(s_q > 0.f) || !(s_k > 0.f) || !(s_v > 0.f) || !(s_p > 0.f) || !std::isfinite(s_q * s_k * s_v / s_p)) return MC_EINVAL;
    if (token_stride < dk || head_stride < dk || (batch > 1 && batch_stride < dk)) return MC_EINVAL;
    if ((int64_t)(L - 1) * token_stride + (int64_t)(heads - 1) * head_stride + dk > (int64_t)INT32_MAX) return MC_EINVAL;
    if (L > (1 << 24) || token_stride >= (1 << 24)) return MC_EINVAL; // kernels use 24-bit multiplies
    if (token_stride % epp != 0 || head_stride % epp != 0 || batch_stride % epp != 0) return MC_EALIGN;
    if (!aligned16(Q_dev) || !aligned16(Km_dev) || !aligned16(Vm_dev) || !aligned16(O_dev)) return MC_EALIGN;
    if (!on_device_of(mask)) return MC_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);

    auto fused = [&](int tile) -> int {           // tile: the kernel's head dimension
        AttnArgs f = {};
        f.real_pieces = dk * qkv_bits / 8 / 16; f.out_cols = dk;
        f.panel_ptr = mask->d_panel_ptr; f.slot_idx = mask->d_slot_idx; f.uniform_vectors = mask->uniform_vectors;
        f.Q = static_cast<const uint8_t *>(Q_dev); f.Km = static_cast<const uint8_t *>(Km_dev);
        f.Vm = static_cast<const uint8_t *>(Vm_dev); f.O = static_cast<float *>(O_dev); f.out_f16 = out_f16;
        f.head_stride = head_stride; f.token_stride = token_stride; f.batch_stride = batch_stride;
        f.in_head_stride = head_stride * qkv_bits / 8; f.in_token_stride = (int)(token_stride * qkv_bits / 8);
        f.in_batch_stride = batch_stride * qkv_bits / 8;
        f.score_scale = s_q * s_k / std::sqrt((float)dk); f.inv_s_p = 1.f / s_p; f.out_scale = s_p * s_v;
        f.heads = heads; f.batch = batch; f.tokens = L;
        // neighbouring heads contiguous inside a token, rows of at most 64 bytes (less than 64 elements where they do not fill the tile): two
        // heads per workgroup can gather 128 bytes per token
        const bool short_rows = dk == 64 || qkv_bits == 4;
        const bool fills = dk == tile && tile <= 128; // (the tile of 192 is a padded one)
        const bool pairs = ((fills && short_rows) || tile == 64) && head_stride == dk && heads % 2 == 0;
        // Pairs by several waves with 16-bit codes take the exponential of entries down to 2^-64 of a row's largest only (FOLDED in the kernel): below that
        // scale of the probabilities, where such entries have codes, one head per workgroup.
        const bool faint = p_bits == 16 && qkv_bits == 8 && !(f.inv_s_p <= FOLDED_MAX_INV_S_P);
        const double avg = mask->P ? (double)(mask->nslots / MC_CHUNK) / mask->P : 0.0;
        // One launch for the panels in `list` (null: all), none of which has more than max_chunks chunks; mean: of theirs.
        auto launch = [&](const int32_t *list, int n_panels, int max_chunks, double mean) -> hipError_t {
            f.panel_list = list; f.P = n_panels;
            f.index_bytes = 4 * std::min(mask->nslots, (int64_t)n_panels * max_chunks * MC_CHUNK);
            // a wave keeps at most 8 chunks of scores in registers: longer panels are shared by 2, 4 or 8 waves
            int wpp = max_chunks > 32 ? 8 : (max_chunks > 16 ? 4 : (max_chunks > 8 ? 2 : 1));
            int hpg;
            if (o.attention_mode == 0) {
                // Halving the gather requests pays once the launch fills the chip (2048 (panel, head) units and
                // more: 13.3 against 15.6 us for 4096 of them; 5.0 against 4.7 us for 128).  Smaller launches get
                // more waves per unit instead, until about 2048 waves are in flight and while at most one of a unit's waves is
                // without a chunk (256 units of 7 chunks: 5.9 us with one wave each, 4.5 us with four; of 3 chunks, dk = 80 - 96, 170 to 438
                // units 6.0 - 6.9 with two, 5.5 - 6.3 with four, dk = 64 2 % less).  All by the chunks of this launch's panels: by the mean of all
                // panels of an unequal mask, whose classes are launched apart, panels of one chunk had four or eight waves and long ones too few.  160 drawn
                // layers on such masks 1.06x in the mean, 0.95 - 1.38 (2 x 2 heads x 1136, dk = 96, nibbles 15.4 -> 11.1 us).  (bench.py --layers times the forms.)
                const int64_t units = (int64_t)n_panels * heads * batch;
                // Two heads, by 240 drawn layers in each form: from 1024 units on where they have 12500 chunks (dk = 64, 1300 to 1700 units of
                // 13 to 18 chunks 1.03 - 1.16 times as fast, below that 0.9 - 1.06), and shorter heads there, too (8 heads x 3384, dk = 48, 9 chunks 35.7 -> 24.2 us,
                // 4 x 3992, 12 chunks 24.3 -> 17.3; 64 layers of 1024 to 4096 units 1.07 in the mean), but for tokens of less than 96 bytes, whose
                // line holds both heads already (0.92 - 1.03), and rows of up to 32 bytes by four waves each (0.94 - 1.08).  Short heads
                // of 4096 units and more from 10000 chunks on (fewer: 0.95 - 1.0).
                const double work = (double)units * mean;
                const int64_t head_bytes = (int64_t)dk * qkv_bits / 8;
                const bool long_enough = units >= 1024 && work >= 12500.0;
                // (From 1152 units on, heads of 48 bytes take more than two chunks a panel: of 1690 layers in every form 22 change, 1.08 times as fast in the
                // mean, 20 of them by more than 2 %, none slower by as much; 8 heads x 2680, 2.5 chunks 11.8 -> 9.4 us; 20 layers of 4160 to 4860 units and 2.0 to
                // 2.33 chunks, less than 10000 in all, 0.98 - 1.13, 1.05 in the mean.  With two chunks and 1152 to 2000 units 0.89 - 1.03.)
                const bool two = fills ? units >= 2048 || long_enough
                                       : (units >= 4096 ? work >= 10000.0 : long_enough && f.in_token_stride >= 96 && (head_bytes > 32 || wpp < 4)) ||
                                             (head_bytes > 32 && units >= 1152 && mean > 2.0);
                // (Not 128 nibbles by four waves each: eight waves of 152 registers are one workgroup a compute unit, a third of its places empty.
                // 2 x 2 heads x 7496, 74 % empty 101.8 -> 74.4 us, 8 x 4800, 75 % 94.7 -> 64.0.)
                hpg = (pairs && two && wpp < 8 && !(fills && tile == 128 && wpp == 4) && !(faint && wpp > 1)) ? 2 : 1;
                // (Rows of 256 bytes, too, where four waves' stages take half a compute unit's LDS: against 1024 waves in flight 46 drawn layers of
                // dk = 144 - 192 1.03 times as fast in the mean, up to 1.23.  4096 waves: 0.98, down to 0.73.)
                if (hpg == 1) while (wpp < 4 && units * wpp * 2 <= 2048 && wpp + 1 <= mean) wpp *= 2;
                // (Eight waves for nine chunks: 225 to 253 units of 9 or 10 1.04 times as fast; 8-bit inputs with 5 to 8 chunks 0.93 - 1.0, nibbles, whose
                // rows take longer to multiply than to fetch, 1.0 - 1.07 from 5 chunks on: three waves without one, too.)
                if (hpg == 1 && wpp == 4 && tile <= 128 && units * 8 <= 2048 && mean >= (qkv_bits == 4 ? 5.0 : 9.0)) wpp = 8;
                // (A few more units than SIMDs, 1024, give some of them two waves and most one; of six chunks on, two waves each: 40 layers of 1026 to 1264 units of 6 to 8
                // chunks 1.0 - 1.18 times as fast, 3 x 3352, dk = 80, 6 chunks 13.9 -> 12.5 us.  Of 3 to 5 chunks 0.95 - 1.08; from 1326 units on 0.8 - 1.04.)
                if (hpg == 1 && wpp == 1 && tile <= 128 && units <= 1280 && mean >= 6.0) wpp = 2;
            } else {
                if (o.attention_mode == 3 && wpp < 2) wpp = 2;
                if (o.attention_mode == 4 && wpp < 4) wpp = 4;
                hpg = (o.attention_mode != 2 && pairs && wpp < 8 && !(faint && wpp > 1)) ? 2 : 1;
            }
            if (fills) return launch_attention_fused(f, hpg, wpp, p_bits, qkv_bits, dk, s);
            return launch_attention_fused_padded(f, hpg, wpp, p_bits, qkv_bits, tile, s);
        };
        // Panels of very different lengths (the longest at least twice the average and more than one wave's
        // worth), automatic mode: one launch per length class, so that short panels are not given the many waves
        // the longest one needs.  Otherwise one launch sized by the longest panel.
        // Small layers, too, are one launch: their classes' launches run one after the other, each with most of the chip idle, and a wave without a chunk
        // costs nothing there.  With panels in three classes and more up to 3000 (panel, head) units, or 1400 where the longest panel takes eight waves and
        // heads are longer than 64 elements; with panels of up to 16 chunks, in two classes, up to 1400.  Of 340 drawn masks both ways, replayed from a
        // graph, the 150 below the lines run 1.5 times as fast in one launch in the mean, 0.99 - 2.55 (2 heads x 1128, 2.1 chunks of up to 18 15.1 -> 6.0 us; 1800 units, dk = 128,
        // 2.4 of up to 19 1.65); of those above one launch takes longer the larger they are (27648 units, dk = 128, 9 of up to 54 chunks 217 us in classes, 478
        // in one), up to 3.4 times, some of up to 5000 units in less time, down to 0.61.  Two classes far apart are on either side, 0.67 - 1.57 below 1500 units.
        const int classes = (mask->class_start[1] > 0) + (mask->class_start[2] > mask->class_start[1]) + (mask->class_start[3] > mask->class_start[2]) +
                            (mask->class_start[4] > mask->class_start[3]);
        const int64_t all_units = (int64_t)mask->P * heads * batch;
        const bool small = classes >= 3 ? all_units <= (mask->max_panel_chunks > 32 && tile > 64 ? 1400 : 3000) : mask->max_panel_chunks <= 16 && all_units <= 1400;
        if (o.attention_mode == 0 && mask->d_class_panels && !small && mask->max_panel_chunks > 8 && mask->max_panel_chunks >= 2.0 * avg) {
            for (int b = 0; b < 4; ++b) {
                const int n = mask->class_start[b + 1] - mask->class_start[b];
                if (n > 0) MC_HIP(launch(mask->d_class_panels + mask->class_start[b], n, b == 3 ? mask->max_panel_chunks : (8 << b), (double)mask->class_chunks[b] / n));
            }
        } else {
            MC_HIP(launch(nullptr, mask->P, mask->max_panel_chunks, avg));
        }
        return MC_OK;
    };
    const int tile = fused_tile(mask, dk, qkv_bits, o);
    if (tile && (tile <= 128 || !use_static)) return fused(tile);
    // the kernel pipeline keeps its intermediates in a workspace (none are needed when nothing is stored)
    const bool with_scores = scores_kernel_waves(mask, heads, dk, qkv_bits, o) == 0;
    const size_t need = attn_layout(heads, mask, p_bits, with_scores).total;
    // sharing long panels between workgroups takes some more room; without it they run whole (same results)
    const size_t need_split = attn_layout(heads, mask, p_bits, with_scores, dk).total;
    const bool split_panels = pipeline_splits(mask, o) && (use_static ? need_split <= STATIC_SCRATCH_BYTES : workspace_bytes >= need_split);
    if (use_static) {
        if (need > STATIC_SCRATCH_BYTES) { // (above 128, too, where the fused kernel would do without: the limit is the layer's, not the form's)
            snprintf(g_detail, sizeof g_detail, "the layer's intermediates need %zu bytes, the library's own array holds %zu",
                     need, STATIC_SCRATCH_BYTES);
            return MC_ENOMEM;
        }
        if (tile) return fused(tile);
        const int rc = static_scratch(&workspace_dev);
        if (rc != MC_OK) return rc;
    } else if (need > 0) {
        if (!workspace_dev) return MC_EINVAL;
        if ((reinterpret_cast<uintptr_t>(workspace_dev) & 255u) != 0) return MC_EALIGN;
        if (workspace_bytes < need) return MC_ENOMEM;
    }
    // the batch items run one after the other through the same workspace
    for (int b = 0; b < batch; ++b) {
        const int64_t ib = (int64_t)b * batch_stride * qkv_bits / 8;
        const int rc = attention_pipeline(static_cast<const uint8_t *>(Q_dev) + ib, static_cast<const uint8_t *>(Km_dev) + ib,
                                          static_cast<const uint8_t *>(Vm_dev) + ib, heads, dk, qkv_bits, p_bits,
                                          head_stride * qkv_bits / 8, token_stride * qkv_bits / 8, head_stride,
                                          token_stride, mask, s_q, s_k, s_v, s_p,
                                          static_cast<uint8_t *>(O_dev) + (int64_t)b * batch_stride * (out_f16 ? 2 : 4),
                                          out_f16, workspace_dev, split_panels, o, s);
        if (rc != MC_OK) return rc;
    }
    return MC_OK;
}
} // namespace

extern "C" size_t mc_attention_workspace_bytes_bits(int heads, const mc_mat *mask, int p_bits)
{
    if (!mask || heads <= 0 || (p_bits != 8 && p_bits != 16)) return 0;
    return attn_layout(heads, mask, p_bits).total;
}

extern "C" size_t mc_attention_workspace_bytes(int heads, const mc_mat *mask)
{
    return mc_attention_workspace_bytes_bits(heads, mask, 8);
}

extern "C" int mc_attention_form(const mc_mat *mask, int dk, int qkv_bits, const mc_options *options)
{
    if (!mask || mask->V != 8 || (qkv_bits != 8 && qkv_bits != 4) || dk <= 0 || dk % (128 / qkv_bits) != 0) return MC_EINVAL;
    mc_options o;
    if (resolve_options(options, &o) != MC_OK) return MC_EINVAL;
    if (fused_tile(mask, dk, qkv_bits, o)) return 0;
    return scores_kernel_waves(mask, 1, dk, qkv_bits, o) ? 1 : 2;
}

extern "C" size_t mc_attention_workspace_needed(int heads, int dk, const mc_mat *mask, int p_bits, const mc_options *options)
{
    if (!mask || heads <= 0 || (p_bits != 8 && p_bits != 16)) return 0;
    mc_options o;
    if (resolve_options(options, &o) != MC_OK) return 0;
    // (8-bit inputs decide here; a 4-bit layer whose rows are not whole pieces then needs what is returned.  Above 128 the figure is
    // the pipeline's whatever the form.)
    if (dk <= 128 && fused_tile(mask, dk, 8, o)) return 0;
    // (the narrowest inputs the layer takes give the smallest rows: whether the scores stay on chip is decided
    // for 8-bit inputs here, which never asks for less than a 4-bit layer needs)
    return attn_layout(heads, mask, p_bits, scores_kernel_waves(mask, heads, dk, 8, o) == 0, pipeline_splits(mask, o) ? dk : 0).total;
}

extern "C" int mc_sparse_attention(const int8_t *Q_dev, const int8_t *Km_dev, const int8_t *Vm_dev, int heads, int L,
                                   int dk, const mc_mat *mask, float s_q, float s_k, float s_v, float s_p,
                                   float *O_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, 1, heads, L, dk, 0, (int64_t)L * dk, dk, mask, 8, 8, s_q, s_k, s_v, s_p,
                          MC_OUT_F32, O_dev, workspace_dev, workspace_bytes, false, nullptr, stream);
}

extern "C" int mc_sparse_attention_strided(const int8_t *Q_dev, const int8_t *Km_dev, const int8_t *Vm_dev, int heads,
                                           int L, int dk, int64_t head_stride, int64_t token_stride,
                                           const mc_mat *mask, float s_q, float s_k, float s_v, float s_p,
                                           float *O_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, 1, heads, L, dk, 0, head_stride, token_stride, mask, 8, 8, s_q, s_k, s_v,
                          s_p, MC_OUT_F32, O_dev, workspace_dev, workspace_bytes, false, nullptr, stream);
}

extern "C" int mc_sparse_attention_bits(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int heads, int L,
                                        int dk, int64_t head_stride, int64_t token_stride, const mc_mat *mask,
                                        int p_bits, int qkv_bits, float s_q, float s_k, float s_v, float s_p,
                                        float *O_dev, void *workspace_dev, size_t workspace_bytes, void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, 1, heads, L, dk, 0, head_stride, token_stride, mask, p_bits, qkv_bits, s_q,
                          s_k, s_v, s_p, MC_OUT_F32, O_dev, workspace_dev, workspace_bytes, false, nullptr, stream);
}

extern "C" int mc_sparse_attention_batched(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int batch,
                                           int heads, int L, int dk, int64_t batch_stride, int64_t head_stride,
                                           int64_t token_stride, const mc_mat *mask, int p_bits, int qkv_bits,
                                           float s_q, float s_k, float s_v, float s_p, float *O_dev,
                                           void *workspace_dev, size_t workspace_bytes, void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, batch, heads, L, dk, batch_stride, head_stride, token_stride, mask, p_bits,
                          qkv_bits, s_q, s_k, s_v, s_p, MC_OUT_F32, O_dev, workspace_dev, workspace_bytes, false, nullptr,
                          stream);
}

extern "C" int mc_sparse_attention_out(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int batch, int heads,
                                       int L, int dk, int64_t batch_stride, int64_t head_stride, int64_t token_stride,
                                       const mc_mat *mask, int p_bits, int qkv_bits, float s_q, float s_k, float s_v,
                                       float s_p, mc_out_type out_type, void *O_dev, void *workspace_dev,
                                       size_t workspace_bytes, void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, batch, heads, L, dk, batch_stride, head_stride, token_stride, mask, p_bits,
                          qkv_bits, s_q, s_k, s_v, s_p, out_type, O_dev, workspace_dev, workspace_bytes, false, nullptr,
                          stream);
}

extern "C" int mc_sparse_attention_ex(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int batch, int heads,
                                      int L, int dk, int64_t batch_stride, int64_t head_stride, int64_t token_stride,
                                      const mc_mat *mask, int p_bits, int qkv_bits, float s_q, float s_k, float s_v,
                                      float s_p, mc_out_type out_type, const mc_options *options, void *O_dev,
                                      void *workspace_dev, size_t workspace_bytes, void *stream)
{
    const mc_options automatic = {};
    return attention_impl(Q_dev, Km_dev, Vm_dev, batch, heads, L, dk, batch_stride, head_stride, token_stride, mask, p_bits,
                          qkv_bits, s_q, s_k, s_v, s_p, out_type, O_dev, workspace_dev, workspace_bytes, false,
                          options ? options : &automatic, stream);
}

extern "C" int mc_sparse_attention_static(const void *Q_dev, const void *Km_dev, const void *Vm_dev, int batch, int heads,
                                          int L, int dk, int64_t batch_stride, int64_t head_stride, int64_t token_stride,
                                          const mc_mat *mask, int p_bits, int qkv_bits, float s_q, float s_k, float s_v,
                                          float s_p, mc_out_type out_type, const mc_options *options, void *O_dev,
                                          void *stream)
{
    return attention_impl(Q_dev, Km_dev, Vm_dev, batch, heads, L, dk, batch_stride, head_stride, token_stride, mask, p_bits,
                          qkv_bits, s_q, s_k, s_v, s_p, out_type, O_dev, nullptr, 0, true, options, stream);
}
