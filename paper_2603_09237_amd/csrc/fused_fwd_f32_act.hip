// The fused forward for fp32 networks, outputs only.
#include "fused_fwd_split.h"

void launch_mlp_fwd_f32_act(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    if (a.split) split_launch_all<false>(a, n_tiles, s);
    else fwd_launch_all<float, false>(a, rt, n_tiles, s);
}
