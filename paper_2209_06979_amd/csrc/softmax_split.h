// Which softmax kernel takes a launch (host code).
#pragma once
#include <stdint.h>

// Pieces of four scores per lane, and waves per panel: one (four panels share a workgroup), or the waves of a workgroup of its own.  No pieces:
// the kernel for panels of any length.
struct SoftmaxSplit { int pieces, waves; };

// longest: scores of the longest panel, padding included.  units: panels of all score sets.  variant: mc_options.softmax_variant.
//
// One wave per panel up to 3072 scores, with as few pieces as it needs; from 1025 scores on workgroups for few panels, whose launch is one
// chain.  us, V = 8, int8 codes, replayed from a graph, against 8 pieces x 2 waves up to 1024 panels, 16 x 1 beyond and 16 x 4 from 4097 scores
// on (the reductions as shuffles through LDS), and as it is:
//   scores   256 panels   1024         4096         32768
//      512   4.1   2.7    4.6   2.7     6.5   4.1    35    17
//     1024   4.2   3.1    4.7   3.3     8.5   6.7    42    32
//     2048   4.4   3.2    5.0   4.0    11.1   9.9    62    60   (256 panels by single waves: 3.8; 1024 by workgroups: 4.7)
//     4096   4.8   3.7    6.1   6.2    17.8  17.3   125   117
//     8192   5.8   4.5   10.8  10.8    32.7  31.8   231   231
//    16384   8.6   8.0   18.2  17.8    68.0  68.1
// A workgroup's fourth piece is nearly empty just above 2048 scores, which a wave of 12 pieces skips (us, workgroups / 12 x 1):
//     2160   640: 4.5  4.4    1024: 5.6  4.7     4096: 13.7  11.1    16384: 41.0  34.7
//     2560   640: 4.6  4.5    1024: 6.0  5.1     4096: 13.7  11.7    16384: 41.5  40.2
//     3040   640: 5.0  4.9    1024: 6.7  6.2     4096: 14.3  12.9    16384: 46.2  47.2
// Up to 4096 scores a workgroup per panel is better while all of them are resident at once (six of four waves a compute unit), a wave of
// 16 pieces beyond, and a workgroup again where panels fill its fourth piece and there are very many (4 x 4 / 16 x 1):
//     3080   1280: 6.7  7.0   1792: 8.2  7.5   2048: 9.3  7.9    4096: 16.1  14.3   16384: 49.5  40.9   24576: 84.0  71.4   32768: 107   93
//     3584   1280: 6.7  7.1   1792: 8.4  7.9   2048: 9.7  8.4    4096: 16.5  15.4   16384: 60.2  48.7   24576: 85.7  84.4   32768: 112  111
//     4096   1280: 6.9  9.5   1792: 9.4  8.9   2048: 10.6  9.6   4096: 17.1  17.3   16384: 62.9  61.8   24576: 92.6  96.2   32768: 117  127
// Up to 8192 scores eight waves of 4 pieces are better than four of 16, but for what four workgroups a compute unit take at once
// and eight waves do not, and for many panels (4 x 8 / 16 x 4):
//     5000   512: 5.9  6.5   768: 7.4  7.4   896: 8.6  8.1   1024: 9.0  8.5   1280: 10.6  11.1   3072: 21.8  21.5   8192: 51.6  49.0   16384: 102   99
//     8192   512: 6.5  7.0   768: 8.2  8.4   896: 10.2  10.0   1024: 11.1  10.7   1280: 13.3  14.5   3072: 25.0  25.5   8192: 68.8  68.9   16384: 127  123
inline SoftmaxSplit softmax_split(int64_t longest, int64_t units, int variant)
{
    const bool few = units <= 512, groups = variant == 1;
    if (variant == 2 || longest > 16384) return {0, 0};
    if (longest > 8192) return {16, 4};
    if (longest > 4096) return units > 4096 || (units > 768 && units <= 1024) ? SoftmaxSplit{16, 4} : SoftmaxSplit{4, 8};
    if (longest > 3072) return groups || units <= 1536 || (units > 20480 && longest > 3584) ? SoftmaxSplit{4, 4} : SoftmaxSplit{16, 1};
    if (longest > 2048) return groups || few ? SoftmaxSplit{4, 4} : SoftmaxSplit{12, 1};
    if (groups || (few && longest > 1024)) return {2, 4};
    return {longest > 1024 ? 8 : longest > 512 ? 4 : 2, 1};
}
