// Launchers of the fused attention kernel for head dimensions 64 and 128 (rows that fill the kernel's tile).
#include "attention_fused.h"

int attention_fused_max_vectors() { return 8 * 8 * 64; }

template <int PB, int QB, int DK> hipError_t launch_pq(const AttnArgs &a, int heads_per_group, int waves_per_panel, hipStream_t s)
{
    if (heads_per_group == 2 && waves_per_panel == 8) return hipErrorInvalidValue;
    if (heads_per_group == 2) {
        // (rows of 128 bytes: one head per workgroup)
        if constexpr (DK == 128 && QB == 8) return hipErrorInvalidValue;
        else {
            if (waves_per_panel == 4) return launch_pairs<2, PB, QB, 4, DK, false>(a, s);
            if (waves_per_panel == 2) return launch_pairs<2, PB, QB, 2, DK, false>(a, s);
            return launch_pairs<2, PB, QB, 1, DK, false>(a, s);
        }
    }
    switch (waves_per_panel) {
    case 8: return launch_pairs<1, PB, QB, 8, DK, false>(a, s);
    case 4: return launch_pairs<1, PB, QB, 4, DK, false>(a, s);
    case 2: return launch_pairs<1, PB, QB, 2, DK, false>(a, s);
    default: return launch_pairs<1, PB, QB, 1, DK, false>(a, s);
    }
}

// waves_per_panel: 1, 2, 4 or 8 waves share the chunks of one (panel, head) (8: one head per workgroup only); a wave
// holds at most 8 chunks of scores in registers, so a panel may have up to 512 * waves_per_panel vectors.
// dk: 64 or 128
hipError_t launch_attention_fused(const AttnArgs &a, int heads_per_group, int waves_per_panel, int p_bits, int qkv_bits,
                                  int dk, hipStream_t s)
{
    if (a.P == 0 || a.heads == 0 || a.batch == 0) return hipSuccess;
    if (dk == 128) {
        if (p_bits == 16) return (qkv_bits == 4) ? launch_pq<16, 4, 128>(a, heads_per_group, waves_per_panel, s)
                                                 : launch_pq<16, 8, 128>(a, heads_per_group, waves_per_panel, s);
        return (qkv_bits == 4) ? launch_pq<8, 4, 128>(a, heads_per_group, waves_per_panel, s)
                               : launch_pq<8, 8, 128>(a, heads_per_group, waves_per_panel, s);
    }
    if (dk != 64) return hipErrorInvalidValue;
    if (p_bits == 16) return (qkv_bits == 4) ? launch_pq<16, 4, 64>(a, heads_per_group, waves_per_panel, s)
                                             : launch_pq<16, 8, 64>(a, heads_per_group, waves_per_panel, s);
    return (qkv_bits == 4) ? launch_pq<8, 4, 64>(a, heads_per_group, waves_per_panel, s)
                           : launch_pq<8, 8, 64>(a, heads_per_group, waves_per_panel, s);
}
