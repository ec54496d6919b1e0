// Shapes of the one-launch forward (fused_fwd.h): waves of a workgroup, LDS, and which networks it may read.  Plain C++,
// so that the host test of the last one compiles it without a GPU toolchain.
#pragma once

#include <stdint.h>

constexpr int kFwdMaxWidth = 512;
constexpr int fwd_waves(int w) { return w <= 256 ? (w + 63) / 64 : w <= 384 ? 6 : 8; }

// row tiles of 16 per workgroup: 1 in fp32 and 2 in bf16, and twice as many for networks of enough waves
constexpr int fwd_low(int es) { return es == 4 ? 1 : 2; }
constexpr bool fwd_has_high(int es, int nw) { return es == 4 ? nw > 1 : nw >= 3; }

inline int fwd_lds_bytes(int es, int O, int W, int L, int rt) {
    const int nw = fwd_waves(W), pitch = (64 * nw * es + 255) / 256 * 256, pitch0 = (O * es + 255) / 256 * 256;
    return 16 * rt * (pitch0 > pitch ? pitch0 : pitch) + nw * 8192 + L * 64 * nw * 4;
}

// Hidden rows are requested up to their end.  The first layer's come as whole super-steps (128 bytes of each row) whatever
// O is, so its last row is followed by less than a super-step of the matrix behind: a hidden layer's always has that much,
// with one hidden layer the output layer's must.  The others keep the layer-by-layer kernels.
inline bool fwd_reads_inside(int es, int W, int L, int out_dim) {
    return W <= kFwdMaxWidth && (L > 1 || out_dim * W >= 128 / es - 1);
}
