// How many (head group, batch item) pairs the fused attention layer works on at a time: host code without a device.
#pragma once
#include "internal.h"

// Lines of 128 bytes that the rows of the busiest of 1, 2, 4, 8 runs of neighbouring pairs touch, against the mean: a gather asks for lines, and an XCD
// that has one head of (L, heads, dk) tensors to itself takes as long as that head's rows cross lines (48 bytes at 96 of 128 do, at 0 do not).
struct PairLines {
    double mean = 0.0, busiest[4] = {1.0, 1.0, 1.0, 1.0};
    // False: no pair differs from the others.  row: bytes of a pair's row, group_stride: from one pair's rows to the next one's.  (Places are of 16-byte pieces within a line; a pattern
    // of eight of them comes round again after eight pairs, so that more than 64 pairs even it out by themselves.)
    bool find(const AttnArgs &a, int64_t pairs, int groups, int row, int64_t group_stride)
    {
        if (pairs % 2 != 0) return false;             // (one pair at a time, whatever their lines)
        if (128 % row == 0 && a.in_token_stride % row == 0) return false;
        if (row % 128 == 0 || pairs > 64 || a.in_token_stride % 128 % 32 != 0) return false; // (the last: every row of a pair in turn at every place)
        int at[8];                                    // lines of four tokens' rows, the first of them at place o
        bool equal = true;
        for (int o = 0; o < 8; ++o) {
            at[o] = 0;
            for (int t = 0; t < 4; ++t) at[o] += ((o * 16 + t * a.in_token_stride) % 128 + row + 127) / 128;
            equal = equal && at[o] == at[0];
        }
        if (equal) return false;
        int run[8] = {}, all = 0;                     // eight runs, whole where they are asked for; eight to a line
        const uintptr_t K = (uintptr_t)a.Km, V = (uintptr_t)a.Vm;
        int64_t item = 0, off = 0;
        for (int p = 0, group = 0, r = 0, left = (int)pairs, n = left; p < n; ++p) {   // (with 64-bit divisions 64 pairs took 0.4 us of host time, not 0.2)
            const int lines = at[(K + off) / 16 % 8] + at[(V + off) / 16 % 8];
            run[r] += lines;
            all += lines;
            off += group_stride;
            if (++group == groups) {
                group = 0;
                off = item += a.in_batch_stride;
            }
            for (left -= 8; left <= 0; left += n) ++r;            // (run 8 p / n)
        }
        mean = all / 8.0 / pairs;
        for (int s = 3; s >= 0; --s) {
            int most = 0;
            for (int k = 0; k < 1 << s; ++k) most = run[k] > most ? run[k] : most;
            busiest[s] = (double)most * (1 << s) / all;
            for (int k = 0; k < 1 << s >> 1; ++k) run[k] = run[2 * k] + run[2 * k + 1];
        }
        return true;
    }
};

// log2 of the pairs worked on at a time, 2^s of them: the s at which the XCDs fetch least from beyond their L2s and the lines they ask L2 for are shared
// out best.  The 8 >> s XCDs of
// a pair fetch its K and V rows (row_bytes), and each its share of the column indices; the share is still there for
// the XCD's next pair if it fits beside a pair's rows into three of L2's four megabytes, or is fetched again for every pair.
// 2^s must divide the number of pairs.  Measured at 1, 2, 4, 8 pairs at a time, 90 % empty, dk = 64, 8-bit codes and inputs:
//   8 x 4 heads x 8192, (heads, L, dk)   217  213  212 (taken)  215 us        16-bit codes 227  219  220 (taken)  226; 4-bit inputs 194  193  191 (taken)  197
//   8 x 4 heads x 8192, (L, heads, dk)   180  179  178.5        177.5 (taken)     4-bit inputs 165  170  168  167.5 (taken)
//   8 x 8 heads x 4096, (heads, L, dk)   122  112  109          108 (taken)   (L, heads, dk) 95.5  92.5  91.5  90 (taken)
//   2 heads x 4096, batch 32             122  113  108          108 (taken)   8 heads x 4096 x 128  27  25  22.1  22.1 (taken)
// and of (L, heads, dk) tensors whose rows cross lines, 8 heads x 3072, 90 % empty:
//   nibbles, dk = 96   15.3  14.7 (taken)  17.1  20.6;   8 bits, dk = 80  18.2  17.0  17.05 (taken)  19.9;   96  19.5  17.9  18.4 (taken)  21.2;
//   112  21.4  20.2 (taken)  21.5  21.6;   48 (four pairs)  12.2  11.9 (taken)  12.7
// A byte more to fetch costs 0.02 - 0.065 ns per kB, since the gather goes on meanwhile; L2 serves 200 lines a ns to this kernel.
inline int pairs_at_a_time(int64_t pairs, double row_bytes, double index_bytes, const PairLines *lines)
{
    constexpr double US_PER_BYTE = 4e-8, LINES_PER_US = 2e5;
    const double asked = lines ? pairs * lines->mean * 2.0 * index_bytes / 4.0 / LINES_PER_US : 0.0;
    int best = 0, plain = 0;
    double least = 0.0, bytes = 0.0, us_plain = 0.0;
    for (int s = 0; s <= 3 && pairs % (1 << s) == 0; ++s) {
        const double share = index_bytes * (1 << s) / 8;
        const double fetched = pairs * row_bytes * (8 >> s) + (row_bytes + share <= 3.0 * (1 << 20) ? 8 * share : pairs * index_bytes);
        const double us = fetched * US_PER_BYTE + (lines ? asked * lines->busiest[s] : 0.0);
        if (s == 0 || us <= least) {
            best = s;
            least = us;
        }
        if (s == 0 || fetched <= bytes) {
            plain = s;
            bytes = fetched;
            us_plain = us;
        }
    }
    return least < us_plain - 0.04 * asked ? best : plain; // (for less than that the estimate is too coarse)
}

// The same for a launch of heads_per_group heads of head_bytes each per workgroup.
inline int attention_pair_shift(const AttnArgs &a, int heads_per_group, int head_bytes)
{
    const int groups = a.heads / heads_per_group, row = heads_per_group * head_bytes, lines = (row + 127) / 128 * 128; // (the L2 holds lines of 128 bytes)
    const int64_t pairs = (int64_t)groups * a.batch;
    PairLines asked;
    const bool differ = asked.find(a, pairs, groups, row, heads_per_group * a.in_head_stride);
    return pairs_at_a_time(pairs, 2.0 * a.tokens * (a.in_token_stride < lines ? a.in_token_stride : lines), (double)a.index_bytes, differ ? &asked : nullptr);
}
