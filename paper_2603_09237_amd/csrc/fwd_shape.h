// Shapes of the one-launch forward (fused_fwd.h): waves of a workgroup, LDS, and which networks it may read.  Plain C++,
// so that the host test of the last one compiles it without a GPU toolchain.
#pragma once

#include <stdint.h>

constexpr int kFwdMaxWidth = 512;
constexpr int fwd_waves(int w) { return w <= 256 ? (w + 63) / 64 : w <= 384 ? 6 : 8; }

inline int fwd_lds_bytes(int es, int O, int W, int L, int rt) {
    const int nw = fwd_waves(W), pitch = (64 * nw * es + 255) / 256 * 256, pitch0 = (O * es + 255) / 256 * 256;
    return 16 * rt * (pitch0 > pitch ? pitch0 : pitch) + nw * 8192 + L * 64 * nw * 4;
}

// Requests come as whole super-steps (128 bytes of each row), and those of a hidden layer always cover the 64 features of
// every wave, so the last row of the last matrix is followed by elements of the output layer: by less than a super-step
// when that matrix is the first layer's, else by 64 NW - W.  Served are the networks whose output layer has that many;
// the others keep the layer-by-layer kernels.  (Rounding W up to a super-step is not enough: fp32 at width 16 requests two.)
inline bool fwd_reads_inside(int es, int W, int L, int out_dim) {
    if (W > kFwdMaxWidth) return false;
    const int head = out_dim * W;
    return head >= (L == 1 ? 128 / es - 1 : 64 * fwd_waves(W) - W);
}
