// Host-side format builder: interchange BCRS (V x 1 blocks) <-> device panel format.
//
// The device format follows the idea of SR-BCRS (paper, Section 4.1): inside a row
// panel the stored vectors are grouped into strides whose length equals the reduction
// depth of the matrix instruction, the last stride is zero-padded, values are stored
// row-major inside a stride, and each panel carries two pointers (aligned start, real
// end).  Here a stride ("chunk") is 64 vectors = one v_mfma_i32_16x16x64_i8, and it is
// cut into 4 sub-strides of 16 vectors because one MFMA lane group consumes 16
// consecutive reduction bytes of one row.
#include "internal.h"

#include <algorithm>
#include <climits>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

namespace {

inline int64_t pad_to_chunk(int64_t n) { return (n + MC_CHUNK - 1) / MC_CHUNK * MC_CHUNK; }

// bytes of one chunk of packed values
// (a 12-bit operand is an int16 array restricted to [-2048, 2047] and is stored like a 16-bit one)
inline int storage_bits(int bits) { return bits == 12 ? 16 : bits; }
inline int64_t chunk_value_bytes(int V, int bits) { return (int64_t)MC_CHUNK * V * storage_bits(bits) / 8; }
inline bool valid_lhs_bits(int b) { return b == 0 || b == 4 || b == 8 || b == 12 || b == 16; }

// signed int8 planes of a 16-bit value: a = 256 * hi + lo, lo in [-128, 127]
inline bool split_balanced(int a, int8_t *hi, int8_t *lo)
{
    int h = (a + 128) >> 8; // arithmetic shift, floor
    int l = a - h * 256;
    *hi = (int8_t)h;
    *lo = (int8_t)l;
    return h >= -128 && h <= 127;
}

// The V elements of interchange vector `vec` in slot `slot` (0..63) of a chunk of packed values (layout: see mc_pack_host).
// The chunk must have been zeroed.  (Vector length and width are constants: an operand's formats write every value up to four times
// over.  With that and the unions below mc_mat_create takes 8.5 ms instead of 11.6 for 3004 x 2900, V = 4, 85 % empty, 16 bits; 4096 x 4096:
// V = 8, 90 % empty 6.8 instead of 7.7; V = 2, half empty 60 instead of 157.)
template <int V, int BITS> struct PutVector {
    int operator()(uint8_t *chunk, int slot, const void *values, int64_t vec) const
    {
        const int g = slot / 16, b = slot % 16;
        if (BITS == 8) {
            const uint8_t *from = static_cast<const uint8_t *>(values) + vec * V;
            uint8_t *to = chunk + g * (16 * V) + b;
            for (int v = 0; v < V; ++v) to[v * 16] = from[v];
        } else if (BITS == 16 || BITS == 12) {
            const int16_t *from = static_cast<const int16_t *>(values) + vec * V;
            uint8_t *to = chunk + g * (32 * V) + b;
            bool fits = true;
            for (int v = 0; v < V; ++v) {
                const int x = from[v];
                int8_t hi, lo;
                fits = split_balanced(x, &hi, &lo) & (BITS == 16 || (x >= -2048 && x <= 2047)) & fits;
                to[v * 16] = (uint8_t)hi;
                to[(V + v) * 16] = (uint8_t)lo;
            }
            if (!fits) return MC_ERANGE;
        } else {
            const uint8_t *from = static_cast<const uint8_t *>(values) + vec * (V / 2);
            uint8_t *to = chunk + g * (8 * V) + (b & 7);
            const int up = b < 8 ? 0 : 4;
            for (int v = 0; v < V; v += 2) {
                to[v * 8] |= (uint8_t)((from[v / 2] & 15) << up);
                to[(v + 1) * 8] |= (uint8_t)((from[v / 2] >> 4) << up);
            }
        }
        return MC_OK;
    }
};

// f(PutVector<V, bits>()) for an operand's V and width (both have been checked)
template <class F> int with_put_vector(int V, int bits, F &&f)
{
    const auto by_V = [&](auto B) {
        constexpr int bits_ = decltype(B)::value;
        switch (V) {
        case 2: return f(PutVector<2, bits_>());
        case 4: return f(PutVector<4, bits_>());
        case 8: return f(PutVector<8, bits_>());
        default: return f(PutVector<16, bits_>());
        }
    };
    switch (bits) {
    case 4: return by_V(std::integral_constant<int, 4>());
    case 8: return by_V(std::integral_constant<int, 8>());
    case 12: return by_V(std::integral_constant<int, 12>());
    default: return by_V(std::integral_constant<int, 16>());
    }
}

// Position of slot s (0..63) of a chunk in the row arrays of the formats below: the two slots one lane of the
// kernel addresses (s and s + 8 inside a sub-stride of 16) are neighbours, so that they travel as one 32-bit word.
inline int64_t chunk_base(int64_t slot) { return slot / MC_CHUNK * MC_CHUNK; }
inline int row_position(int s) { return (s / 16) * 16 + (s % 8) * 2 + (s % 16) / 8; }

} // namespace

// The builders below exist in two forms: the exported ones take the vector lengths of the interchange format
// (2, 4, 8); the *_wide ones also take 16 for 4- and 8-bit values, which only the library's own merged copy of
// an operand uses (see mc_merge_host): sixteen rows fill the MFMA's row operand completely.
static bool valid_V_wide(int V, int lhs_bits)
{
    return V == 2 || V == 4 || V == 8 || (V == 16 && (lhs_bits == 4 || lhs_bits == 8));
}

extern "C" int mc_layout_query(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, mc_layout *out)
{
    return V == 16 ? MC_EINVAL : mc_layout_query_wide(M, K, V, lhs_bits, row_ptr, out);
}

int mc_layout_query_wide(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, mc_layout *out)
{
    if (!row_ptr || !out) return MC_EINVAL;
    if (M <= 0 || K <= 0) return MC_EINVAL;
    if (!valid_V_wide(V, lhs_bits)) return MC_EINVAL;
    if (M % V != 0) return MC_EINVAL;
    if (!valid_lhs_bits(lhs_bits)) return MC_EINVAL;
    const int P = M / V;
    if (row_ptr[0] != 0) return MC_EINVAL;
    int64_t nslots = 0;
    for (int p = 0; p < P; ++p) {
        const int64_t n = (int64_t)row_ptr[p + 1] - row_ptr[p];
        if (n < 0 || n > K) return MC_EINVAL;
        nslots += pad_to_chunk(n);
    }
    if (nslots > (int64_t)INT32_MAX - MC_CHUNK) return MC_EINVAL;
    out->P = P;
    out->nvec = row_ptr[P];
    out->nslots = nslots;
    out->vals_bytes = lhs_bits ? (nslots / MC_CHUNK) * chunk_value_bytes(V, lhs_bits) : 0;
    return MC_OK;
}

extern "C" int mc_pack_host(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx,
                            const void *values, int32_t *panel_ptr, int32_t *slot_idx, void *slot_vals)
{
    return V == 16 ? MC_EINVAL : mc_pack_host_wide(M, K, V, lhs_bits, row_ptr, col_idx, values, panel_ptr, slot_idx, slot_vals);
}

int mc_pack_host_wide(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx,
                      const void *values, int32_t *panel_ptr, int32_t *slot_idx, void *slot_vals)
{
    mc_layout lay;
    int rc = mc_layout_query_wide(M, K, V, lhs_bits, row_ptr, &lay);
    if (rc != MC_OK) return rc;
    if (!panel_ptr || (lay.nslots && !slot_idx) || (lay.nvec && !col_idx)) return MC_EINVAL;
    const bool with_vals = lhs_bits != 0 && values != nullptr;
    if (with_vals && lay.vals_bytes && !slot_vals) return MC_EINVAL;

    // pattern
    int64_t slot0 = 0;
    for (int p = 0; p < lay.P; ++p) {
        const int64_t lo = row_ptr[p], n = (int64_t)row_ptr[p + 1] - lo;
        panel_ptr[2 * p] = (int32_t)slot0;
        panel_ptr[2 * p + 1] = (int32_t)(slot0 + n);
        int32_t prev = -1;
        for (int64_t i = 0; i < n; ++i) {
            const int32_t c = col_idx[lo + i];
            if (c <= prev || c >= K) return MC_EINVAL;
            slot_idx[slot0 + i] = c;
            prev = c;
        }
        for (int64_t i = n; i < pad_to_chunk(n); ++i) slot_idx[slot0 + i] = prev; // n > 0 here
        slot0 += pad_to_chunk(n);
    }
    if (!with_vals) return MC_OK;

    std::memset(slot_vals, 0, (size_t)lay.vals_bytes);
    uint8_t *dst = static_cast<uint8_t *>(slot_vals);
    const int64_t cbytes = chunk_value_bytes(V, lhs_bits);
    return with_put_vector(V, lhs_bits, [&](auto put) -> int {
        for (int p = 0; p < lay.P; ++p) {
            const int64_t lo = row_ptr[p], n = (int64_t)row_ptr[p + 1] - lo;
            const int64_t s0 = panel_ptr[2 * p];
            for (int64_t i = 0; i < n; ++i) {
                const int64_t s = s0 + i;
                const int bad = put(dst + (s / MC_CHUNK) * cbytes, (int)(s % MC_CHUNK), values, lo + i);
                if (bad != MC_OK) return bad;
            }
        }
        return MC_OK;
    });
}

extern "C" int mc_unpack_host(int M, int K, int V, int lhs_bits, const int32_t *panel_ptr,
                              const int32_t *slot_idx, const void *slot_vals, int32_t *row_ptr,
                              int32_t *col_idx, void *values)
{
    if (M <= 0 || K <= 0 || (V != 2 && V != 4 && V != 8) || M % V) return MC_EINVAL;
    if (!valid_lhs_bits(lhs_bits)) return MC_EINVAL;
    if (!panel_ptr || !row_ptr) return MC_EINVAL;
    const int P = M / V;
    const uint8_t *src = static_cast<const uint8_t *>(slot_vals);
    const int64_t cbytes = lhs_bits ? chunk_value_bytes(V, lhs_bits) : 0;
    const bool with_vals = lhs_bits != 0 && slot_vals != nullptr && values != nullptr;
    int64_t out = 0;
    row_ptr[0] = 0;
    for (int p = 0; p < P; ++p) {
        const int64_t s0 = panel_ptr[2 * p], n = (int64_t)panel_ptr[2 * p + 1] - s0;
        if (n < 0 || s0 % MC_CHUNK) return MC_EINVAL;
        for (int64_t i = 0; i < n; ++i, ++out) {
            const int64_t s = s0 + i;
            col_idx[out] = slot_idx[s];
            if (!with_vals) continue;
            const uint8_t *chunk = src + (s / MC_CHUNK) * cbytes;
            const int g = (int)(s % MC_CHUNK) / 16, b = (int)(s % 16);
            for (int v = 0; v < V; ++v) {
                const int64_t e = out * V + v;
                if (lhs_bits == 8) {
                    static_cast<uint8_t *>(values)[e] = chunk[g * (16 * V) + v * 16 + b];
                } else if (lhs_bits == 16 || lhs_bits == 12) {
                    const int hi = (int8_t)chunk[g * (32 * V) + v * 16 + b];
                    const int l8 = (int8_t)chunk[g * (32 * V) + 16 * V + v * 16 + b];
                    static_cast<int16_t *>(values)[e] = (int16_t)(hi * 256 + l8);
                } else {
                    const uint8_t byte = chunk[g * (8 * V) + v * 8 + (b & 7)];
                    const int nib = (b < 8) ? (byte & 15) : (byte >> 4);
                    uint8_t *o = &static_cast<uint8_t *>(values)[e >> 1];
                    if (e & 1) *o = (uint8_t)((*o & 0x0F) | (nib << 4));
                    else *o = (uint8_t)((*o & 0xF0) | nib);
                }
            }
        }
        row_ptr[p + 1] = (int32_t)out;
    }
    return MC_OK;
}

// ---- K-blocked variant of the format -------------------------------------------------------
// A host-side format of the public interface that no kernel here reads (the resident SpMM has its own, see mc_resident_pack):
// blocks of MC_KBLOCK consecutive rows of the dense operand; the vectors of a panel are additionally grouped by the K-block their column
// falls in, and each (panel, block) list is padded to whole chunks on its own, so that every
// chunk only names rows of one block (as 16-bit row numbers inside that block).
extern "C" int mc_blocked_query(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx,
                                mc_blocked_layout *out)
{
    mc_layout lay;
    int rc = mc_layout_query(M, K, V, lhs_bits, row_ptr, &lay);
    if (rc != MC_OK) return rc;
    if (!out || (lay.nvec && !col_idx)) return MC_EINVAL;
    const int nblk = (K + MC_KBLOCK - 1) / MC_KBLOCK;
    int64_t nchunks = 0;
    for (int p = 0; p < lay.P; ++p) {
        int64_t i = row_ptr[p];
        const int64_t end = row_ptr[p + 1];
        int32_t prev = -1;
        for (int b = 0; b < nblk; ++b) {
            int64_t n = 0;
            while (i < end && col_idx[i] < (int64_t)(b + 1) * MC_KBLOCK) {
                if (col_idx[i] <= prev || col_idx[i] >= K) return MC_EINVAL;
                prev = col_idx[i];
                ++i; ++n;
            }
            nchunks += (n + MC_CHUNK - 1) / MC_CHUNK;
        }
        if (i != end) return MC_EINVAL; // a column at or beyond K
    }
    if (nchunks * MC_CHUNK > (int64_t)INT32_MAX - MC_CHUNK) return MC_EINVAL;
    out->nblk = nblk;
    out->nchunks = nchunks;
    out->vals_bytes = lhs_bits ? nchunks * chunk_value_bytes(V, lhs_bits) : 0;
    return MC_OK;
}

extern "C" int mc_pack_blocked_host(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx,
                                    const void *values, int32_t *blk_ptr, uint16_t *blk_rows, void *blk_vals,
                                    int32_t *blk_src)
{
    mc_blocked_layout bl;
    int rc = mc_blocked_query(M, K, V, lhs_bits, row_ptr, col_idx, &bl);
    if (rc != MC_OK) return rc;
    if (!blk_ptr || (bl.nchunks && (!blk_rows || !blk_src))) return MC_EINVAL;
    const bool with_vals = lhs_bits != 0 && values != nullptr;
    if (with_vals && bl.vals_bytes && !blk_vals) return MC_EINVAL;
    if (with_vals) std::memset(blk_vals, 0, (size_t)bl.vals_bytes);
    uint8_t *dst = static_cast<uint8_t *>(blk_vals);
    const int64_t cbytes = lhs_bits ? chunk_value_bytes(V, lhs_bits) : 0;
    const int P = M / V;
    int64_t chunk = 0;
    for (int p = 0; p < P; ++p) {
        int64_t i = row_ptr[p];
        const int64_t end = row_ptr[p + 1];
        for (int b = 0; b < bl.nblk; ++b) {
            blk_ptr[(int64_t)p * bl.nblk + b] = (int32_t)chunk;
            int64_t n = 0;
            int last_row = 0;
            while (i < end && col_idx[i] < (int64_t)(b + 1) * MC_KBLOCK) {
                const int64_t slot = chunk * MC_CHUNK + n;
                last_row = col_idx[i] - b * MC_KBLOCK;
                blk_rows[chunk_base(slot) + row_position((int)(slot % MC_CHUNK))] = (uint16_t)last_row;
                blk_src[slot] = (int32_t)i;
                if (with_vals) {
                    rc = with_put_vector(V, lhs_bits, [&](auto put) -> int { return put(dst + (slot / MC_CHUNK) * cbytes, (int)(slot % MC_CHUNK), values, i); });
                    if (rc != MC_OK) return rc;
                }
                ++i; ++n;
            }
            const int64_t npad = (n + MC_CHUNK - 1) / MC_CHUNK * MC_CHUNK;
            for (int64_t k = n; k < npad; ++k) { // padded slots: a row of this block, zero values, no source vector
                blk_rows[chunk_base(chunk * MC_CHUNK + k) + row_position((int)(k % MC_CHUNK))] = (uint16_t)last_row;
                blk_src[chunk * MC_CHUNK + k] = -1;
            }
            chunk += npad / MC_CHUNK;
        }
    }
    blk_ptr[(int64_t)P * bl.nblk] = (int32_t)chunk;
    return MC_OK;
}

// ---- LDS-ordered copy ------------------------------------------------------------------------
// For the kernel that keeps whole rows of a column tile of the dense operand in LDS (internal.h has the layout).
// 160 KB hold 2560 rows of 64 bytes or 5120 of 32; more rows than that come in equal blocks.
void mc_resident_query(int K, int P, const int32_t *row_ptr, const int32_t *col_idx, ResidentLayout *out)
{
    out->nt = K <= 2560 ? 4 : 2;
    const int most = 10240 / out->nt;
    out->nblk = (K + most - 1) / most;
    out->block_rows = ((K + out->nblk - 1) / out->nblk + 15) / 16 * 16;
    int64_t nchunks = 0;
    for (int p = 0; p < P; ++p) {
        if (out->nblk == 1) {
            nchunks += std::max(1, (row_ptr[p + 1] - row_ptr[p] + MC_CHUNK - 1) / MC_CHUNK);
            continue;
        }
        const int32_t *i = col_idx + row_ptr[p], *end = col_idx + row_ptr[p + 1];
        for (int b = 0; b < out->nblk; ++b) {
            const int32_t *e = std::lower_bound(i, end, (b + 1) * out->block_rows);
            nchunks += std::max<int64_t>(1, (e - i + MC_CHUNK - 1) / MC_CHUNK);
            i = e;
        }
    }
    out->nchunks = nchunks;
}

int mc_resident_pack(int K, int V, int lhs_bits, int P, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                     const ResidentLayout &lay, int32_t *ptr, uint8_t *recs, int32_t *src, uint32_t *ends)
{
    const int64_t cbytes = chunk_value_bytes(V, lhs_bits), rec_chunks = resident_rec_chunks(lay.nblk, V, lhs_bits), rbytes = rec_chunks * (2 * MC_CHUNK + cbytes);
    const bool pairs = rec_chunks == 2;
    return with_put_vector(V, lhs_bits, [&](auto put) -> int {
        std::vector<int32_t> place;                 // interchange vector of each place of a list, -1: empty
        std::vector<int32_t> extra[16];             // vectors whose residue has more of them than the list has sets
        int64_t chunk = 0;
        for (int p = 0; p < P; ++p) {
            const int32_t *i = col_idx + row_ptr[p], *end = col_idx + row_ptr[p + 1];
            for (int b = 0; b < lay.nblk; ++b) {
                ptr[(int64_t)p * lay.nblk + b] = (int32_t)chunk;
                const int32_t *e = lay.nblk == 1 ? end : std::lower_bound(i, end, (b + 1) * lay.block_rows);
                const int row0 = b * lay.block_rows, nrows = std::min(K - row0, lay.block_rows);
                const int nch = std::max(1, (int)((e - i + MC_CHUNK - 1) / MC_CHUNK)), nsets = nch * 4;
                // A set is the 16 rows that half a wave reads at once; place 16*set + residue.  The k-th row of a residue
                // goes to set k; what exceeds the number of sets fills the places left over, one of a residue per set.
                place.assign((size_t)nsets * 16, -1);
                int count[16] = {0};
                for (const int32_t *c = i; c < e; ++c) {
                    const int res = (*c - row0) & 15, at = count[res]++;
                    if (at < nsets) place[(size_t)at * 16 + res] = (int32_t)(c - col_idx);
                    else extra[res].push_back((int32_t)(c - col_idx));
                }
                int left = 0;                           // vectors in `extra`
                for (int res = 0; res < 16; ++res) left += std::max(0, count[res] - nsets);
                for (int st = 0; st < nsets && left > 0; ++st) {
                    int res = 0;
                    for (int t = 0; t < 16; ++t) {
                        if (st < count[t]) continue;    // (taken)
                        while (res < 16 && extra[res].empty()) ++res;
                        if (res == 16) break;
                        place[(size_t)st * 16 + t] = extra[res].back();
                        extra[res].pop_back();
                        ++res;
                        --left;
                    }
                }
                for (int st = 0; st < nsets && left > 0; ++st) { // (a last resort: several of one residue in a set)
                    for (int t = 0; t < 16 && left > 0; ++t) {
                        if (place[(size_t)st * 16 + t] >= 0) continue;
                        int res = 0;
                        while (extra[res].empty()) ++res;
                        place[(size_t)st * 16 + t] = extra[res].back();
                        extra[res].pop_back();
                        --left;
                    }
                }
                for (int st = 0; st < nsets; ++st) {
                    const int64_t c = chunk + st / 4, second = pairs ? c & 1 : 0; // (second chunk of its record)
                    uint8_t *rec = recs + (pairs ? c >> 1 : c) * rbytes, *vals = rec + (pairs ? 4 * MC_CHUNK : 2 * MC_CHUNK) + second * (cbytes / 4);
                    const int pair = (st % 4) / 2, h = st % 2;   // lane groups 2*pair, 2*pair + 1; slots 8h .. 8h + 7 of each
                    for (int t = 0; t < 16; ++t) {
                        const int slot = (2 * pair + t / 8) * 16 + 8 * h + t % 8;
                        const int32_t from = place[(size_t)st * 16 + t];
                        const int row = from >= 0 ? col_idx[from] - row0 : (t < nrows ? t : 0);
                        const int at = row_position(slot);
                        reinterpret_cast<uint16_t *>(rec)[pairs ? (at / 2 * 2 + second) * 2 + at % 2 : at] = (uint16_t)((row >> 4) * 16 * lay.nt + (row & 15));
                        src[c * MC_CHUNK + slot] = from;
                        if (from >= 0) {
                            // (two chunks: a group of 16 slots of the other one after each of this one's)
                            const int rc = put(vals + (pairs ? slot / 16 * (cbytes / 4) : 0), slot, values, from);
                            if (rc != MC_OK) return rc;
                        }
                    }
                }
                chunk += nch;
                if (lay.nblk == 1) ends[(chunk - 1) / 32] |= 1u << ((chunk - 1) % 32);
                i = e;
            }
        }
        ptr[(int64_t)P * lay.nblk] = (int32_t)chunk;
        return MC_OK;
    });
}

// ---- merged panels ----------------------------------------------------------------------------
// `group` consecutive panels of V rows become one panel of V * group rows whose stored vectors sit at the
// union of the panels' columns; a panel that has no vector at a column of the union contributes zeros there
// (explicit zeros are legal inside stored vectors).  The product with a dense matrix is unchanged, the rows
// of the dense operand named by a column are fetched once for all the panels of a group instead of once per
// panel that holds it, and the MFMA's 16-row operand fills up.
namespace {
// The union of a few panels' columns: a bit per column, and a bit per word of those.
class ColumnUnion {
    std::vector<uint64_t> bits, words;
public:
    explicit ColumnUnion(int K) : bits((size_t)K / 64 + 1), words((size_t)K / 4096 + 1) {}
    void add(int32_t c)
    {
        bits[(size_t)c >> 6] |= (uint64_t)1 << (c & 63);
        words[(size_t)c >> 12] |= (uint64_t)1 << ((c >> 6) & 63);
    }
    // f(word number, its bits) in ascending order; the union is empty afterwards
    template <class F> void drain(F &&f)
    {
        for (size_t i = 0; i < words.size(); ++i)
            for (uint64_t w = words[i]; w; w &= w - 1) {
                const size_t at = i * 64 + (size_t)__builtin_ctzll(w);
                f(at, bits[at]);
                bits[at] = 0;
            }
        std::fill(words.begin(), words.end(), 0);
    }
};

int merged_query(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx, int group, mc_merged_layout *out)
{
    mc_layout lay;
    int rc = mc_layout_query(M, K, V, lhs_bits, row_ptr, &lay);
    if (rc != MC_OK) return rc;
    if (!out || (lay.nvec && !col_idx)) return MC_EINVAL;
    if (group < 2 || (V * group != 8 && V * group != 16)) return MC_EINVAL;
    if (V * group == 16 && lhs_bits != 4 && lhs_bits != 8) return MC_EINVAL;
    const int Pm = (lay.P + group - 1) / group;
    int64_t nvec = 0;
    ColumnUnion columns(K);
    for (int sp = 0; sp < Pm; ++sp) {
        const int p0 = sp * group, p1 = std::min(p0 + group, lay.P);
        for (int p = p0; p < p1; ++p) {
            int32_t prev = -1;
            for (int64_t i = row_ptr[p]; i < row_ptr[p + 1]; ++i) { // ascending, inside [0, K)
                if (col_idx[i] <= prev || col_idx[i] >= K) return MC_EINVAL;
                prev = col_idx[i];
                columns.add(prev);
            }
        }
        columns.drain([&](size_t, uint64_t bits) { nvec += __builtin_popcountll(bits); });
    }
    if (nvec > (int64_t)INT32_MAX - MC_CHUNK) return MC_EINVAL;
    out->group = group;
    out->P = Pm;
    out->nvec = nvec;
    return MC_OK;
}

template <int VB> struct Share { typedef uint8_t type; };
template <> struct Share<2> { typedef uint16_t type; };
template <> struct Share<4> { typedef uint32_t type; };
template <> struct Share<8> { typedef uint64_t type; };

// VB: bytes of one panel's share of a merged vector (0: pattern only)
template <int VB, int group> void merge(int P, int K, const int32_t *row_ptr, const int32_t *col_idx, const uint8_t *src, int Pm, int32_t *m_row_ptr,
                                        int32_t *m_col_idx, uint8_t *dst, int32_t *m_src)
{
    ColumnUnion columns(K);
    int64_t out = 0;
    m_row_ptr[0] = 0;
    for (int sp = 0; sp < Pm; ++sp) {
        const int p0 = sp * group, np = std::min(group, P - p0);
        int32_t at[group], end[group];             // (panels beyond the last are empty)
        for (int g = 0; g < group; ++g) {
            at[g] = g < np ? row_ptr[p0 + g] : 0;
            end[g] = g < np ? row_ptr[p0 + g + 1] : 0;
            for (int32_t i = at[g]; i < end[g]; ++i) columns.add(col_idx[i]);
        }
        columns.drain([&](size_t word, uint64_t bits) {
            for (; bits; bits &= bits - 1, ++out) {
                const int32_t c = (int32_t)(word * 64) + __builtin_ctzll(bits);
                m_col_idx[out] = c;
                for (int g = 0; g < group; ++g) { // (no branches: whether a panel has the column is anybody's guess)
                    const int32_t i = at[g] < end[g] ? at[g] : 0;
                    const int here = (at[g] < end[g]) & (col_idx[i] == c);
                    m_src[out * group + g] = here ? i : -1;
                    at[g] += here;
                    if (VB) {
                        typename Share<VB>::type x;
                        std::memcpy(&x, src + (int64_t)i * VB, sizeof x);
                        x &= (typename Share<VB>::type)-here;
                        std::memcpy(dst + (out * group + g) * VB, &x, sizeof x);
                    }
                }
            }
        });
        m_row_ptr[sp + 1] = (int32_t)out;
    }
}
} // namespace

extern "C" int mc_merged_query(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx, int group,
                               mc_merged_layout *out)
{
    try {
        return merged_query(M, K, V, lhs_bits, row_ptr, col_idx, group, out);
    } catch (const std::bad_alloc &) {
        return MC_ENOMEM;
    }
}

extern "C" int mc_merge_host(int M, int K, int V, int lhs_bits, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                             int group, int32_t *m_row_ptr, int32_t *m_col_idx, void *m_values, int32_t *m_src)
{
    mc_merged_layout ml;
    int rc = mc_merged_query(M, K, V, lhs_bits, row_ptr, col_idx, group, &ml);
    if (rc != MC_OK) return rc;
    if (!m_row_ptr || (ml.nvec && (!m_col_idx || !m_src))) return MC_EINVAL;
    const bool with_vals = lhs_bits != 0 && values != nullptr && m_values != nullptr;
    const int vb = with_vals ? V * storage_bits(lhs_bits) / 8 : 0; // bytes of one panel's share of a merged vector
    const auto run = [&](auto VB) {
        const auto of = [&](auto G) {
            merge<decltype(VB)::value, decltype(G)::value>(M / V, K, row_ptr, col_idx, static_cast<const uint8_t *>(values), ml.P, m_row_ptr,
                                                           m_col_idx, static_cast<uint8_t *>(m_values), m_src);
        };
        if (group == 2) of(std::integral_constant<int, 2>());
        else if (group == 4) of(std::integral_constant<int, 4>());
        else of(std::integral_constant<int, 8>());
        return MC_OK;
    };
    try {
        switch (vb) {
        case 0: return run(std::integral_constant<int, 0>());
        case 1: return run(std::integral_constant<int, 1>());
        case 2: return run(std::integral_constant<int, 2>());
        case 4: return run(std::integral_constant<int, 4>());
        case 8: return run(std::integral_constant<int, 8>());
        default: return MC_EINVAL;                 // (shares of 16 bytes are not merged)
        }
    } catch (const std::bad_alloc &) {
        return MC_ENOMEM;
    }
}
