// The fused forward for fp32 networks, saving what the backward pass reads.
#include "fused_fwd_split.h"

void launch_mlp_fwd_f32_save(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    if (a.split) split_launch_all<true>(a, n_tiles, s);
    else fwd_launch_all<float, true>(a, rt, n_tiles, s);
}
