// The fused forward for bf16 networks, saving what the backward pass reads.
#include "fused_fwd.h"

void launch_mlp_fwd_bf16_save(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    fwd_launch_all<bf16_t, true>(a, rt, n_tiles, s);
}
