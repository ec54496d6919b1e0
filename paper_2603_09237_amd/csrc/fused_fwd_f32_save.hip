// The fused forward for fp32 networks, saving what the backward pass reads.
#include "fused_fwd.h"

void launch_mlp_fwd_f32_save(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    fwd_launch_all<float, true>(a, rt, n_tiles, s);
}
