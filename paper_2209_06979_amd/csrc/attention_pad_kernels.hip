// Launchers of the fused attention kernel for head dimensions that do not fill its tile of 64 or 128
// elements, and of up to 192 (any multiple of 16; of 32 for 4-bit inputs): the missing pieces of
// every row read as zeros (see PAD in attention_fused.h); one head per workgroup, or two of less than 64 elements.
#include "attention_fused.h"

namespace {
template <int PB, int QB, int DK> hipError_t launch_padded(const AttnArgs &a, int waves_per_panel, hipStream_t s)
{
    switch (waves_per_panel) {
    case 8:
        if constexpr (DK == 192) return hipErrorInvalidValue; // (such panels go to the pipeline)
        else return launch_pairs<1, PB, QB, 8, DK, true>(a, s);
    case 4: return launch_pairs<1, PB, QB, 4, DK, true>(a, s);
    case 2: return launch_pairs<1, PB, QB, 2, DK, true>(a, s);
    default: return launch_pairs<1, PB, QB, 1, DK, true>(a, s);
    }
}

template <int PB, int QB> hipError_t launch_padded_64(const AttnArgs &a, int heads_per_group, int waves_per_panel, hipStream_t s)
{
    if (heads_per_group == 1) return launch_padded<PB, QB, 64>(a, waves_per_panel, s);
    if (waves_per_panel == 8) return hipErrorInvalidValue;
    if (waves_per_panel == 4) return launch_pairs<2, PB, QB, 4, 64, true>(a, s);
    if (waves_per_panel == 2) return launch_pairs<2, PB, QB, 2, 64, true>(a, s);
    return launch_pairs<2, PB, QB, 1, 64, true>(a, s);
}
} // namespace

// heads_per_group: 2 only with a tile of 64 and heads that are contiguous inside a token.  tile: 64, 128 or 192, the kernel's head dimension; a.real_pieces * 16 bytes is what a row really has
// (fewer, with 192 at most, than tile * qkv_bits / 8), a.out_cols the real head dimension.
hipError_t launch_attention_fused_padded(const AttnArgs &a, int heads_per_group, int waves_per_panel, int p_bits, int qkv_bits, int tile, hipStream_t s)
{
    if (a.P == 0 || a.heads == 0 || a.batch == 0) return hipSuccess;
    if (a.real_pieces <= 0 || a.out_cols <= 0) return hipErrorInvalidValue;
    if (tile == 192 ? (a.real_pieces * 16 > tile * qkv_bits / 8 || a.out_cols > tile)
                    : (a.real_pieces * 16 >= tile * qkv_bits / 8 || a.out_cols >= tile))
        return hipErrorInvalidValue;
    if (heads_per_group == 2 && tile != 64) return hipErrorInvalidValue;
    if (tile == 192) {
        if (p_bits == 16) return (qkv_bits == 4) ? launch_padded<16, 4, 192>(a, waves_per_panel, s) : launch_padded<16, 8, 192>(a, waves_per_panel, s);
        return (qkv_bits == 4) ? launch_padded<8, 4, 192>(a, waves_per_panel, s) : launch_padded<8, 8, 192>(a, waves_per_panel, s);
    }
    if (tile == 128) {
        if (p_bits == 16) return (qkv_bits == 4) ? launch_padded<16, 4, 128>(a, waves_per_panel, s) : launch_padded<16, 8, 128>(a, waves_per_panel, s);
        return (qkv_bits == 4) ? launch_padded<8, 4, 128>(a, waves_per_panel, s) : launch_padded<8, 8, 128>(a, waves_per_panel, s);
    }
    if (tile != 64) return hipErrorInvalidValue;
    if (p_bits == 16) return (qkv_bits == 4) ? launch_padded_64<16, 4>(a, heads_per_group, waves_per_panel, s) : launch_padded_64<16, 8>(a, heads_per_group, waves_per_panel, s);
    return (qkv_bits == 4) ? launch_padded_64<8, 4>(a, heads_per_group, waves_per_panel, s) : launch_padded_64<8, 8>(a, heads_per_group, waves_per_panel, s);
}
