// The fused forward for bf16 networks, outputs only.
#include "fused_fwd.h"

void launch_mlp_fwd_bf16_act(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    fwd_launch_all<bf16_t, false>(a, rt, n_tiles, s);
}
