// Shapes of the one-launch forward (fused_fwd.h): waves of a workgroup, LDS, and which networks it may read.  Plain C++,
// so that the host test of the last one compiles it without a GPU toolchain.
#pragma once

#include <stdint.h>

constexpr int kFwdMaxWidth = 512;
constexpr int fwd_waves(int w) { return w <= 256 ? (w + 63) / 64 : w <= 384 ? 6 : 8; }

// row tiles of 16 per workgroup: 1 in fp32 and 2 in bf16, and twice as many for bf16 networks of enough waves and for the fp32
// networks that tiles of split operands (below) do not always serve
constexpr int fwd_low(int es) { return es == 4 ? 1 : 2; }
constexpr bool fwd_has_high(int es, int nw) { return es == 4 ? nw == 2 : nw >= 3; }

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

// fp32 networks of width 256 and less (fused_fwd_split.h): waves of 32 features; three planes of bf16 parts, rows in pitches that
// the swizzle knows.  The last super-steps of a hidden row run on into the next rows, behind the last row into the output layer's
// matrix, which is at least as long as a row.
constexpr int kSplitMaxWidth = 256;
constexpr int split_pitch(int k) { return k <= 32 ? 64 : (k * 2 + 127) / 128 * 128; }
constexpr int split_waves(int w) { return w <= 128 ? (w + 31) / 32 : w <= 160 ? 5 : w <= 192 ? 6 : 8; }
constexpr int split_most(int nw) { return nw <= 2 ? 1 : nw == 5 || nw == 6 ? 3 : 2; }  // most 32-row blocks of a tile
inline int split_lds_bytes(int O, int W, int L, int rb) {
    const int nw = split_waves(W), p0 = split_pitch(O), p1 = split_pitch(32 * nw);
    return 3 * 32 * rb * (p0 > p1 ? p0 : p1) + nw * 4096 + L * 32 * nw * 4;
}
