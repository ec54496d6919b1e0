// The fused forward for fp32 networks, outputs only.
#include "fused_fwd.h"

void launch_mlp_fwd_f32_act(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    fwd_launch_all<float, false>(a, rt, n_tiles, s);
}
