// Shapes of the one-launch forward (fused_fwd.h): waves of a workgroup, LDS, which networks it may read, and which tiles a
// call takes.  Plain C++, so that the host tests of the last two compile it without a GPU toolchain.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define MORLAX_HD __host__ __device__
#else
#define MORLAX_HD
#endif

// Division of numbers below 2^31 by one divisor d, exact, as a product and a shift: with s = ceil(log2 d) and mul = floor(2^(31 +
// s) / d) + 1 the excess mul d - 2^(31 + s) lies in (0, d], d <= 2^s, so that m mul / 2^(31 + s) is above m / d by less than 1 / d.
struct RowDiv {
    uint32_t mul;
    int32_t sh;
    MORLAX_HD uint32_t quotient(uint32_t m) const { return (uint32_t)(((uint64_t)m * mul) >> sh); }
};
inline RowDiv row_div(int32_t d) {
    int s = 0;
    while ((int64_t)1 << s < d) ++s;
    return {(uint32_t)(((uint64_t)1 << (31 + s)) / (uint32_t)d + 1), 31 + s};
}

constexpr int kFwdMaxWidth = 512;
constexpr int fwd_waves(int w) { return w <= 256 ? (w + 63) / 64 : w <= 384 ? 6 : 8; }

// row tiles of 16 per workgroup: 1 in fp32 and 2 in bf16, and twice as many for bf16 networks of enough waves
constexpr int fwd_low(int es) { return es == 4 ? 1 : 2; }
constexpr bool fwd_has_high(int es, int nw) { return es == 2 && nw >= 3; }
// the row tiles of the kernel that runs where `rt` are asked for: the launch and its count of workgroups both take this
constexpr int fwd_compiled(int es, int nw, int rt) { return fwd_has_high(es, nw) && rt == 2 * fwd_low(es) ? rt : fwd_low(es); }

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

// The tiles of a one-launch forward of `rows` rows per preference: row tiles of 16 a workgroup (0: not this kernel, but the one
// that multiplies four times the rows per fetched weight for tall selections of width 512 or 256, `tall_kernel`, or the
// layer-by-layer GEMMs) and, on split operands, their 32-row blocks.  The lines are measured ones (saving variant, three hidden
// layers, preferences x rows; us).
struct FwdPlan { int rt, split; };
inline FwdPlan fwd_plan(int es, int W, int L, int O, int out_dim, int P, int64_t rows, int cus, bool tall_kernel) {
    const int nw = fwd_waves(W);
    if (!fwd_reads_inside(es, W, L, out_dim)) return {0, 0};
    auto tiles = [&](int r) { return (int64_t)P * ((rows + 16 * r - 1) / (16 * r)); };
    auto fits = [&](int r) { return fwd_lds_bytes(es, O, W, L, r) <= 160 * 1024; };
    if (!fits(fwd_low(es))) return {0, 0};
    if (es == 2) {
        // W 512: 64 x 512 107 tall, 137 here; 16 x 1024 (128 tall tiles) 72 and 59.  W 256: 64 x 1024 71 and 87, 64 x 512
        // (256 tall tiles) 52 and 42
        if ((W == 512 && tiles(8) >= 192) || (W == 256 && tiles(8) >= 384))
            if (tall_kernel) return {0, 0};
        if (nw == 8 && !tall_kernel && tiles(4) >= 512) return {0, 0};
        if (nw == 6 && tiles(4) >= 512) return {0, 0};  // W 384: 64 x 700 141 and 145, 64 x 2048 327 and 408, 16 x 700 54 and 46
        // tiles of 64 rows once 32 would leave more than two rounds of workgroups: W 512 16 x 1024 59 against 63, 64 x 128
        // 59 against 38; W 144 64 x 700 55 against 63, 16 x 700 28 against 25; W 48 and 128 (2, 4 tiles at a time on a CU) never
        return {fwd_has_high(2, nw) && tiles(2) >= (nw == 3 ? 1024 : 512) && fits(4) ? 4 : 2, 0};
    }
    if (W <= kSplitMaxWidth) {
        // Tiles of 32, 64 or 96 rows on split operands (fused_fwd_split.h), of 16 on the fp32 instructions while there are too few
        // for more than the length of one tile's chain to matter.  16 and 32 rows, plain / saving: W 256 16 x 128 24 / 26 and
        // 24 / 27, 64 x 128 35 / 38 and 28 / 33; W 160 16 x 20 20 / 20 and 18 / 20; W 128 16 x 128 14 / 15.5 and 14 / 16, 64 x 128
        // 20 / 23 and 14 / 18; W 64 64 x 128 11 / 13 and 11 / 13.4, 16 x 700 11.8 / 14.8 and 14.8 / 18.7, 16 x 2048 19 / 24 and 17 / 22;
        // W 32 16 x 700 12.3 / 13.7 and 12.5 / 14.8, 16 x 2048 19 / 21 and 13 / 18
        const int snw = split_waves(W);
        auto fits_split = [&](int rb) { return rb <= split_most(snw) && split_lds_bytes(O, W, L, rb) <= 160 * 1024; };
        // One hidden layer, whose products are few: W 128 10 x 1065 10.7 / 12.5 and 11.9 / 14.6, W 144 5 x 141 10.9 / 10.6 and 10.9 / 11.6;
        // W 208 107 x 119 17 / 19 and 11 / 15
        const int least_tiles = snw <= 2 || (L == 1 && snw <= 4) ? 704 : snw == 5 && L > 1 ? 0 : 128;
        // Up to 64 features, one or two waves a workgroup split all of a tile's observations: worth it only while the first layer is
        // short beside the hidden ones.  Times of 16-row tiles over split ones, plain / saving, 704 to 8192 tiles of 32 rows: W 32, one
        // hidden layer, O 33 0.98 - 1.14 / 0.97 - 1.10, O 64 0.86 - 0.96 / 0.88 - 0.94; two, O 64 1.05 - 1.35 / 0.96 - 1.16, O 100 0.96 -
        // 1.14 / 0.87 - 1.04, O 200 0.90 - 1.16 / 0.77 - 1.03, O 513 0.53 - 0.70 / 0.67 - 0.80; three, O 128 1.01 - 1.19 / 0.92 - 1.06.
        // From 1536 tiles on, W 64, two, O 33 1.06 - 1.18 / 1.03 - 1.14, O 64 0.97 - 0.99 / 0.93 - 0.98 and from 4096 1.05 - 1.10 / 1.00 -
        // 1.08, O 200 0.86 - 0.96 / 0.87 - 0.90; three, O 64 1.18 - 1.33 / 1.11 - 1.20, O 128 1.03 - 1.06 / 0.94 - 1.07.  W 48, a quarter
        // of whose products are padding, two, O 33 0.96 - 1.08 / 0.89 - 1.00 and from 6144 1.12 - 1.15 / 0.99 - 1.03; three, O 64 1.18 -
        // 1.20 / 1.03 - 1.07
        const bool long_first = O > (snw == 1 ? 48 : 32) * L;
        if (snw <= 2 && long_first && fits_split(1)) return {1, 0};
        if (snw == 2 && (!fits_split(1) || tiles(2) < (W < 64 && L < 3 ? 6144 : O > 24 * L ? 4096 : 1536))) return {1, 0};
        if (tiles(2) < least_tiles || !fits_split(1)) return {tiles(1) < 1408 ? 1 : 0, 0};
        int split = 1;
        if (snw <= 2) return {2, 1};
        // W 65 to 128, several tiles at a time on a CU, 32 and 64 rows: 16 x 300 14 / 17 and 17 / 22, 16 x 700 20 / 25 and 18 / 25,
        // 64 x 2048 108 / 167 and 89 / 155
        if (snw <= 4) split = tiles(2) > cus && fits_split(2) ? 2 : 1;
        // above, one tile at a time on a CU: whichever takes fewest rounds of them, in the time one tile of 32, 64 or 96 rows
        // takes (W 160 18, 24.5 and 34 us for three layers; W 256 24 and 34).  W 160, 32, 64 and 96 rows: 16 x 700 34, 24, 33; 10 x 1850
        // 51, 48, 34; 10 x 3700 84, 71, 66; 16 x 2048 67, 47, 65; 64 x 2048 268, 189, 197
        const int cost[] = {30, snw == 8 ? 43 : 41, 56};
        int64_t least = INT64_MAX;
        for (int rb = 1; rb <= 3 && snw > 4; ++rb) {
            const int64_t c = (tiles(2 * rb) + cus - 1) / cus * cost[rb - 1];
            if (fits_split(rb) && c < least) { split = rb; least = c; }
        }
        return {2 * split, split};
    }
    // wider ones, tiles of 16 rows while there is a CU for each: 16 rows and the layer-by-layer GEMMs, W 512 16 x 256 56 / 60 and
    // 78 / 81, 64 x 128 109 / 118 and 87 / 93; W 384 64 x 64 43 / 47 and 65 / 68, 64 x 128 79 / 85 and 71 / 74; W 272 64 x 64
    // 45 / 46 and 51 / 55, 16 x 700 117 / 123 and 75 / 77
    // (one hidden layer: W 512 25 x 198 28 / 32 and 37 / 38)
    return {tiles(1) <= (L == 1 ? 768 : 256) ? 1 : 0, 0};
}
