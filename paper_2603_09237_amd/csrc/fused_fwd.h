// Fused target-network forward (paper Sec. III-C, rollout and update phases): observations -> every hidden layer ->
// output layer with tanh, sampling and log-density, in one launch.
//
// A workgroup of NW waves carries ROWS = 16 RT rows of one preference through every layer.  The activations of the
// tile live in LDS (16-byte chunks XOR-swizzled by the row) and are rewritten in place layer after layer; HBM sees the
// observations, the outputs and, in the saving variant, the stores of h and act'(z) the backward pass reads.
// Wave w owns output features [64 w, 64 w + 64) of every layer for all rows of the tile, so its slice of W_l(p) is
// used by no other wave.  It travels a super-step (a 128-byte line of each of the 64 rows, 8 KB) at a time: requested
// into registers D super-steps ahead, across layer ends, then through 8 KB of LDS of the wave's own -- no barrier stands
// between a request and its use.
//
// Why through LDS: an MFMA operand wants consecutive lanes on consecutive rows, and the vector cache looks addresses up
// four lanes at a time -- fetched that way from a row-major matrix that is four lookups per 64 bytes.  A loop that only
// requests three 512 x 512 matrices, one workgroup of eight waves a CU and 16 KB a wave in flight, takes 46 us that way (16
// bytes per clock and CU) and 19 us with eight lanes to a line, while the caches serve the weights (32 workgroups on 16
// networks; 256 on 8: 47 and 20 us).  With every CU on weights of its own the way from memory bounds both: 59 and 63 us; the
// largest policies are there (128 preferences x 128 rows of 4 x 512, both networks in turn, whose 422 MB of weights come from
// memory: 56.7 us a network, 3.7 TB/s, 62.7 before the ring was filled ahead of the first layer; one network again and again, most
// of its 211 MB out of the memory-side cache: 48 to 49, 4.4 TB/s, and 53 to 55).  (Copying the matrices into fragment order first, as the kernel for tall selections does, is a launch of 87
// us at that size.)
//
// bf16 products are 32x32x16 in the contraction order of the kernels that serve taller selections of the same network
// (k_mlp_fused_fwd: `perm`, chunks jj and 4 + jj of a line together, bias first; the tiled GEMMs: ascending, bias last;
// k_first_fwd_narrow: one fused multiply-add after the other), so that an output does not depend on how many rows are
// asked for.  fp32 products are 16x16x4, whose smaller tiles reach more CUs; the launcher takes them while tiles are few
// (fwd_plan), else those of fused_fwd_split.h or the layer-by-layer GEMMs.
#pragma once

#include <atomic>

#include "fwd_shape.h"
#include "mlp_device.h"

struct FwdNet {  // the network family of a call
    const void* theta_mat;   // [P][mat_len]: W_0 [W][O], W_1 .. [W][W] back to back, then the output layer
    const float* theta_vec;  // [P][vec_len]: W biases a layer, then the output layer's
    int64_t mat_len, vec_len;
    int64_t head_mat_off, head_vec_off, logsig_off;
    int32_t out_dim, tanh_cols;  // leading output columns that are squashed by tanh (the actor's means)
    int32_t adim, sig_state;     // action width; 1: log sigma = output columns [adim, 2 adim) of the same row
    int32_t M, tiles_m;          // rows per preference, row tiles per preference
    RowMap rm;
    float* out;        // time-major [.., N, out_dim]
    float* saved_out;  // saving: compact [P][M][OUT_PITCH]
    const float* eps;  // actor with sampling: noise, and the two outputs below
    float* act;
    float* logp;
    char* H;   // saving: h of layer l at H + l * lstride, [P][Mp][ldh]
    char* G;   // saving: act'(z), likewise
    char* x0;  // saving, optional: the selected observations in the GEMM input type, [P][Mp][ldx]
};

struct FwdArgs {
    const float* x;  // observations, time-major rows of O values
    FwdNet net;
    int32_t L, O, W, act;
    int32_t perm, narrow;  // bf16: contraction order, first layer by multiply-adds (see above)
    int32_t split;         // fp32: 32-row blocks of a tile of fused_fwd_split.h, 0: tiles of this file's kernel
    int32_t Mp, ldh, ldx;  // saving: rows per preference and row lengths of the compact buffers
    int64_t lstride;       // bytes
};

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));  // (HIP's uint4 keeps arrays of it out of registers)
typedef u32x4_t chunk2_t __attribute__((aligned(2)));          // 16 bytes at any element boundary

// Piece c of a row of O >= VE values: VE of them, zeros beyond O.  obs_get requests the VE values that end with the row where the
// piece runs past it, obs_place moves them down.  (With whole pieces and single values in branches of their own the compiler
// waits for one piece before it requests the next.)
template <int NQ>
__device__ inline void obs_get(u32x4_t (&q)[NQ], const float* row, int c, int O) {
    constexpr int VE = 4 * NQ;
    typedef u32x4_t word_t __attribute__((aligned(4)));
    const float* at = row + (VE * c + VE <= O ? VE * c : O - VE);
#pragma unroll
    for (int e = 0; e < NQ; ++e) q[e] = *reinterpret_cast<const word_t*>(at + 4 * e);
}
template <int VE>
__device__ inline void obs_place(float (&v)[VE], const u32x4_t (&q)[VE / 4], int c, int O) {
#pragma unroll
    for (int e = 0; e < VE; ++e) v[e] = __uint_as_float(q[e >> 2][e & 3]);
    const bool end = VE * c + VE > O, in = VE * c < O;
    const int d = (VE - O % VE) % VE;  // (the same for every row)
    if (d)
#pragma unroll
        for (int b = 1; b < VE; b *= 2) {
            const bool move = end && (d & b);
#pragma unroll
            for (int e = 0; e < VE; ++e) v[e] = move ? (e + b < VE ? v[e + b < VE ? e + b : 0] : 0.f) : v[e];
        }
#pragma unroll
    for (int e = 0; e < VE; ++e) v[e] = in ? v[e] : 0.f;
}

// super-steps of W requested ahead: what the registers leave room for, as long as it divides those of a hidden layer
// (fp32: a super-step's products take so long that two cover the latency)
constexpr int fwd_depth(int es, int nw, int rt) {
    if (es == 4) return 2;
    return nw % 2 == 0 ? 2 : nw == 3 && rt <= 2 ? 3 : 1;
}

// a value the compiler can no longer trace back to its source: address arithmetic derived from it stays
// where it is written instead of being hoisted into registers held across the products
__device__ inline int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ inline int swap_bits23(int i) { return (i & 0x13) | ((i & 4) << 1) | ((i & 8) >> 1); }

// activation and derivative, rounded as the kernels that serve taller selections round them
enum { kActTanh = 0, kActSiluFused = 1, kActSiluPlain = 2 };
template <typename T, int MODE>
__device__ inline void fwd_act(float z, float& h, float& g) {
    if (MODE == kActTanh || sizeof(T) == 2) {
        act_pair<T, MODE == kActTanh ? 0 : 1, MODE == kActSiluFused>(z, h, g);
    } else {
#pragma clang fp contract(off)
        const float s = __builtin_amdgcn_rcpf(1.f + __expf(-z)), z1 = 1.f + z;
        h = z * s;
        const float d = z1 - h;
        g = s * d;
    }
}

// WHOLE: the waves' features are the network's, W = 64 NW (as a condition at run time: 31.6 against 29.1 us for
// one step of 32 preferences x 256 rows of width 256, the two kinds of requests waiting for each other's registers).
// fp32 tiles stay within the 168 registers of three waves a SIMD: with 169 the update step of 10
// preferences x 3700 rows of width 160 took 1.48 ms, 1.42 now.
template <typename T, bool SAVE, int NW, int RT, bool WHOLE>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 ? 3 : 2) void k_mlp_fwd(FwdArgs a) {
    constexpr int ES = sizeof(T), VE = 16 / ES;
    constexpr bool B32 = ES == 2;    // 32x32 products
    constexpr int KS = 8 * VE;       // contraction indices of a super-step: a 128-byte line of every W row
    constexpr int WP = 64 * NW;      // features the waves cover; those beyond W are zero
    constexpr int S1 = WP / KS;      // super-steps of a hidden layer
    constexpr int PITCH = (WP * ES + 255) / 256 * 256;
    constexpr int ROWS = 16 * RT;
    constexpr int D = fwd_depth(ES, NW, RT);
    // The ring is filled with the tile's other first requests, where tall saving tiles do not wait for each other's stores: ahead
    // of the first layer and behind it, 20 preferences x 850 rows of 3 x 256, saving, 29.6 and 27.3 us, 128 x 128 of 4 x 512
    // 79.8 and 78.6 (acting, one network again and again, ahead: 51.6 -> 46.1)
    constexpr bool EARLY = !SAVE || RT <= 2;
    static_assert(S1 % D == 0, "the ring of requests wraps at layer ends");
    extern __shared__ __align__(16) unsigned char dlds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const FwdNet& net = a.net;
    const int p = tile / net.tiles_m, m0 = (tile % net.tiles_m) * ROWS;
    const int O = a.O, W = WHOLE ? WP : a.W, L = a.L;
    const bool perm = B32 && a.perm;
    const char* Wp = reinterpret_cast<const char*>(net.theta_mat) + (int64_t)p * net.mat_len * ES;
    const float* bp = net.theta_vec + (int64_t)p * net.vec_len;
    const int n0 = (O + KS - 1) / KS;  // super-steps of the first layer
    const int pitch0 = (n0 * 128 + 255) & ~255;
    const int tile_bytes = ROWS * (pitch0 > PITCH ? pitch0 : PITCH);
    unsigned char* wst = dlds + tile_bytes + wave * 8192;  // this wave's super-step of W; in an epilogue, its store patch
    float* sbias = reinterpret_cast<float*>(dlds + tile_bytes + NW * 8192);  // [L][WP]

    // W in LDS: 64 feature rows of eight 16-byte chunks, chunk c of row R at position c ^ ((R >> 1) & 7), so that the
    // fragment reads of 16 lanes (16 rows, one chunk) cover all banks.  Request b of lane l is position l & 7 of row
    // 8 b + (l >> 3).  Features beyond W repeat the last row (zeroed in the epilogue).  `left`: elements from here to the
    // end of a hidden row (a multiple of VE), chunks beyond which are zeros.
    auto load_w = [&](u32x4_t (&w)[8], const char* base, int ld, int left) __attribute__((always_inline)) {
        const int ol = opaque(lane);  // (formed here: addresses held across the products would cost them registers)
        const int q0 = ((ol & 7) ^ ((ol >> 4) & 3)) * 16;  // chunk of even b; odd b: the other half of the line
        if constexpr (WHOLE) {
            const uint32_t row = (uint32_t)((64 * wave + (ol >> 3)) * ld) * ES;
#pragma unroll
            for (int b = 0; b < 8; ++b)
                w[b] = *reinterpret_cast<const chunk2_t*>(base + (int64_t)(8 * b * ld) * ES + (row + (uint32_t)(q0 ^ (64 * (b & 1)))));
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {  // even b, odd b
                const int q = q0 ^ (64 * h);
                if (q < left * ES) {
#pragma unroll
                    for (int b = h; b < 8; b += 2) {
                        const int f = 64 * wave + 8 * b + (ol >> 3);
                        w[b] = *reinterpret_cast<const chunk2_t*>(base + ((uint32_t)((f < W ? f : W - 1) * ld) * ES + (uint32_t)q));
                    }
                } else {
#pragma unroll
                    for (int b = h; b < 8; b += 2) w[b] = u32x4_t{0, 0, 0, 0};
                }
            }
        }
    };
    auto store_w = [&](const u32x4_t (&w)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 8; ++b) *reinterpret_cast<u32x4_t*>(wst + b * 1024 + lane * 16) = w[b];
    };
    u32x4_t w0[8];
    const bool narrow = B32 && a.narrow;
    auto load_w0 = [&]() __attribute__((always_inline)) {
        if (narrow) {  // (O <= 32) lane = feature: its whole row
            const int f = 64 * wave + lane;
            const char* row = Wp + (uint32_t)((f < W ? f : W - 1) * O) * ES;
#pragma unroll
            for (int b = 0; b < 4; ++b) w0[b] = *reinterpret_cast<const chunk2_t*>(row + 16 * b);
        } else {
            load_w(w0, Wp, O, KS);
        }
    };
    // The first layer's last super-step runs past the end of the rows into the next ones, or into the matrix behind
    // (fwd_reads_inside: the launcher checks that there is enough of it).  The observations it meets there are zero, but an
    // infinite or undefined weight of another row would make a NaN of them, so those elements are zeroed: `kept` of register
    // e of request b are not.  bf16: by masks formed here, while the requests are on their way (behind them: 32.5 against
    // 29.1 us for one step of 32 preferences x 256 rows of width 256); in fp32 the masks' registers would spill.
    auto kept = [&](int l, int b, int e) __attribute__((always_inline)) {
        return O - (n0 - 1) * KS - (((l & 7) ^ ((l >> 4) & 3) ^ (4 * (b & 1))) * VE + e * (4 / ES));
    };
    u32x4_t keep[2];
    if constexpr (B32) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int n = kept(lane, h, e);
                keep[h][e] = n > 1 ? 0xffffffffu : n > 0 ? 0xffffu : 0u;
                asm volatile("" : "+v"(keep[h][e]));
            }
    }
    // requests of the hidden layers; past the last layer the cursor repeats a valid one, so that every super-step has
    // the same number of loads in flight
    u32x4_t wf[D][8];
    int cl = 1, cs = 0;
    auto fetch = [&](u32x4_t (&w)[8]) __attribute__((always_inline)) {
        load_w(w, Wp + ((int64_t)W * O + (int64_t)(cl - 1) * W * W) * ES + cs * 128, W, W - cs * KS);
        if (++cs == S1) {
            cs = 0;
            cl = cl + 1 < L ? cl + 1 : cl;
        }
    };
    auto fill = [&]() __attribute__((always_inline)) {
        if (L > 1) {
#pragma unroll
            for (int u = 0; u < D; ++u) fetch(wf[u]);
        }
    };

    // What the tile starts from is requested together, what is needed first ahead of the rest: observations, biases (a register
    // load later on would stand behind the ring's requests), W_0, the ring.  us, as a loop of pieces with two divisions each,
    // the biases layer by layer behind it, and so, one network again and again: acting, 128 preferences x 128 rows of 4 x 512 51.4 and
    // 45.6 (both networks in turn 62.7 and 56.7 each), 32 x 256 of 3 x 256 14.2 and 13.6, 64 x 6000 of 3 x 64 with 120 observations 126 and 78; saving, 38 x 850 of 3 x 256 47.8 and 43.9.
    {
        constexpr int NT = 64 * NW, NB = 4;  // layers whose biases come along
        constexpr int G = 4 * RT >= 4 * NW ? 4 : (4 * RT + NW - 1) / NW;  // pieces a thread requests together: 128 observations in bf16, 64 in fp32
        // 2^sh pieces of VE values a row, those behind the last super-step skipped, those behind the observations zero
        const int np = 8 * n0, nc = ((O + 7) & ~7) / VE, sh = 32 - __builtin_clz(np - 1), n_id = ROWS << sh;
        const int mlim = SAVE ? a.Mp - m0 : 0;
        const int bf = (int)threadIdx.x < W ? threadIdx.x : W - 1;
        // the observations in the GEMM input type, zero-filled to whole steps; rows past the end repeat the last row (their
        // outputs are never stored)
        auto obs_row = [&](int r) __attribute__((always_inline)) {
            return a.x + (uint32_t)net.rm.row(p, m0 + r < net.M ? m0 + r : net.M - 1) * (uint32_t)O;  // (the tensor stays below 4 GiB)
        };
        auto load_x = [&](u32x4_t (&v)[G][VE / 4], int first) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = first + g * NT + (int)threadIdx.x, id = i < n_id ? i : n_id - 1;
                obs_get(v[g], obs_row(id >> sh), id & ((1 << sh) - 1), O);
            }
        };
        auto put_piece = [&](const float (&v)[VE], int r, int c) __attribute__((always_inline)) {
            const uint4 q = pack_chunk<T>(v);
            *reinterpret_cast<uint4*>(dlds + r * pitch0 + ((c ^ (r & 15)) * 16)) = q;
            if (SAVE && net.x0 && r < mlim && c < nc)
                *reinterpret_cast<uint4*>(net.x0 + (((int64_t)p * a.Mp + m0 + r) * a.ldx + VE * c) * ES) = q;
        };
        auto put_x = [&](u32x4_t (&v)[G][VE / 4], int first) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int id = first + g * NT + (int)threadIdx.x, r = id >> sh, c = id & ((1 << sh) - 1);
                float w[VE];
                obs_place(w, v[g], c, O);
                if (id < n_id && c < np) put_piece(w, r, c);
            }
        };
        u32x4_t v[G][VE / 4];
        int first = 0;
        if (O >= VE) {
            for (; first + G * NT < n_id; first += G * NT) {
                load_x(v, first);
                put_x(v, first);
            }
            load_x(v, first);
        }
        float bv[NB];
#pragma unroll
        for (int l = 0; l < NB; ++l) bv[l] = bp[(l < L ? l : L - 1) * W + bf];
        __builtin_amdgcn_sched_barrier(0);
        load_w0();
        if (EARLY) fill();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int l = 0; l < NB; ++l)
            if (l < L) sbias[l * WP + threadIdx.x] = bv[l];
        for (int l = NB; l < L; ++l) sbias[l * WP + threadIdx.x] = bp[l * W + bf];
        if (O >= VE) {
            put_x(v, first);
        } else {  // rows shorter than a piece, element by element
            for (int r = threadIdx.x; r < ROWS; r += NT) {
                const float* row = obs_row(r);
                float w[VE];
#pragma unroll
                for (int e = 0; e < VE; ++e) w[e] = e < O ? row[e < O ? e : O - 1] : 0.f;
                put_piece(w, r, 0);
                for (int c = 1; c < np; ++c) {
                    const float zero[VE] = {};
                    put_piece(zero, r, c);
                }
            }
        }
    }
    if (narrow) {  // W_0 transposed: [input][feature] of the wave
        const uint32_t wq[16] = {w0[0].x, w0[0].y, w0[0].z, w0[0].w, w0[1].x, w0[1].y, w0[1].z, w0[1].w,
                                 w0[2].x, w0[2].y, w0[2].z, w0[2].w, w0[3].x, w0[3].y, w0[3].z, w0[3].w};
#pragma unroll
        for (int i = 0; i < 32; ++i)
            reinterpret_cast<uint16_t*>(wst)[i * 64 + lane] = (uint16_t)(wq[i >> 1] >> (16 * (i & 1)));
    }

    // accumulators.  bf16: 32-row block i, feature block j: lane (lr, lg) holds row 32 i + lr, features 32 j + 16 h + 8 lg
    // + u in element 8 h + u.  fp32: row tile i, feature block b: row 16 i + ln, features 16 b + 4 kg + e in element e.
    constexpr int NI = B32 ? RT / 2 : RT, NJ = B32 ? 2 : 4;
    typedef typename std::conditional<B32, float16_t, float4_t>::type acc_t;
    acc_t acc[NI][NJ];
    const int lr = B32 ? (lane & 31) : (lane & 15), lg = B32 ? lane >> 5 : lane >> 4;  // row in the tile, lane group
    auto piece_feature = [&](int q, int g) __attribute__((always_inline)) { return B32 ? 16 * q + 8 * g : 16 * q + 4 * g; };
    auto init_acc = [&](int l, bool zero) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b4 = 0; b4 < VE / 4; ++b4) {
                float4 b = *reinterpret_cast<const float4*>(sbias + l * WP + 64 * wave + piece_feature(q, lg) + 4 * b4);
                if (zero) b = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    if constexpr (B32) {
                        acc[i][q >> 1][8 * (q & 1) + 4 * b4] = b.x; acc[i][q >> 1][8 * (q & 1) + 4 * b4 + 1] = b.y;
                        acc[i][q >> 1][8 * (q & 1) + 4 * b4 + 2] = b.z; acc[i][q >> 1][8 * (q & 1) + 4 * b4 + 3] = b.w;
                    } else {
                        acc[i][q] = float4_t{b.x, b.y, b.z, b.w};
                    }
                }
            }
    };
    // super-step s of a layer; W rows in an order that gives a lane eight consecutive features (bf16)
    const int wrow = B32 ? swap_bits23(lr) : lr;
    auto products = [&](const u32x4_t (&wreg)[8], int s, int pitch) __attribute__((always_inline)) {
        store_w(wreg);
        const unsigned char* ws = wst + wrow * 128;
        const unsigned char* as = dlds + lr * pitch;
        const int sw = (wrow >> 1) & 7, x = lr & 15;
        if constexpr (B32) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = perm ? 4 * lg + v : 2 * v + lg;
                uint4 w[2], fa[NI];
#pragma unroll
                for (int j = 0; j < 2; ++j) w[j] = *reinterpret_cast<const uint4*>(ws + j * 4096 + ((c ^ sw) * 16));
#pragma unroll
                for (int i = 0; i < NI; ++i) fa[i] = *reinterpret_cast<const uint4*>(as + i * 32 * pitch + (((8 * s + c) ^ x) * 16));
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) Mma32<T>::run(w[j], fa[i], acc[i][j]);
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = 4 * h + lg;
                uint4 w[4], fa[RT];
#pragma unroll
                for (int b = 0; b < 4; ++b) w[b] = *reinterpret_cast<const uint4*>(ws + b * 2048 + ((c ^ sw) * 16));
#pragma unroll
                for (int i = 0; i < RT; ++i) fa[i] = *reinterpret_cast<const uint4*>(as + i * 16 * pitch + (((8 * s + c) ^ x) * 16));
#pragma unroll
                for (int e = 0; e < 4; ++e)  // the four products of a chunk, one round over all accumulators each
#pragma unroll
                    for (int i = 0; i < RT; ++i)
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(chunk_f32(w[b], e), chunk_f32(fa[i], e), acc[i][b], 0, 0, 0);
            }
        }
    };
    auto epilogue = [&](int l, bool add_bias, auto act_tag) __attribute__((always_inline)) {
        constexpr int MODE = decltype(act_tag)::value;
        const int mlim = SAVE ? a.Mp - m0 : 0;
        const int el = opaque(lane), er = B32 ? (el & 31) : (el & 15), eg = B32 ? el >> 5 : el >> 4;
        const int64_t at = (int64_t)l * a.lstride + ((int64_t)p * a.Mp + m0) * a.ldh * ES;
        char* Hl = SAVE ? net.H + at : nullptr;
        char* Gl = SAVE ? net.G + at : nullptr;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = (B32 ? 32 : 16) * i + er;
            if (B32) __builtin_amdgcn_sched_barrier(0);  // one row block's temporaries at a time: no spills
            uint4 gq[4], hq[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int f = 64 * wave + piece_feature(q, eg);
                float v[8], g[8];
#pragma unroll
                for (int u = 0; u < VE; ++u) v[u] = B32 ? acc[i][q >> 1][8 * (q & 1) + u] : acc[i][q & 3][u & 3];
                if (B32 && add_bias) {
#pragma unroll
                    for (int u = 0; u < VE; ++u) v[u] += sbias[l * WP + f + u];
                }
#pragma unroll
                for (int u = 0; u < VE; ++u) fwd_act<T, MODE>(v[u], v[u], g[u]);
                if (!WHOLE && f >= W) {
#pragma unroll
                    for (int u = 0; u < VE; ++u) v[u] = g[u] = 0.f;
                }
                hq[q] = pack_chunk<T>(v);
                gq[q] = pack8(g, (const typename GradT<T>::type*)nullptr).lo;
                *reinterpret_cast<uint4*>(dlds + row * PITCH + (((f / VE) ^ (er & 15)) * 16)) = hq[q];
                if (SAVE && !B32) {  // four lanes' pieces of a row are 64 contiguous bytes
                    if (row < mlim && (WHOLE || f < a.ldh)) {
                        const uint32_t o = (uint32_t)(row * a.ldh + f) * ES;
                        *reinterpret_cast<uint4*>(Gl + o) = gq[q];
                        *reinterpret_cast<uint4*>(Hl + o) = hq[q];
                    }
                }
            }
            if (SAVE && B32) {  // through the wave's room for W, so that a store instruction writes whole 128-byte row segments
#pragma unroll
                for (int arr = 0; arr < 2; ++arr) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<uint4*>(wst + er * 128 + (((2 * q + eg) ^ (er & 7)) * 16)) = arr ? hq[q] : gq[q];
                    __builtin_amdgcn_wave_barrier();
                    char* dst = arr ? Hl : Gl;
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const int prow = it * 8 + (el >> 3), pc = el & 7, f = 64 * wave + pc * 8;
                        const uint4 u = *reinterpret_cast<const uint4*>(wst + prow * 128 + ((pc ^ (prow & 7)) * 16));
                        if (32 * i + prow < mlim && (WHOLE || f < a.ldh))
                            *reinterpret_cast<uint4*>(dst + (uint32_t)((32 * i + prow) * a.ldh + f) * ES) = u;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    };
    auto finish_layer = [&](int l, bool add_bias) __attribute__((always_inline)) {
        __syncthreads();  // every wave has read the layer's input for the last time
        if (a.act == 0) epilogue(l, add_bias, std::integral_constant<int, kActTanh>{});
        else if (B32 && (perm || (narrow && l == 0))) epilogue(l, add_bias, std::integral_constant<int, kActSiluFused>{});
        else epilogue(l, add_bias, std::integral_constant<int, kActSiluPlain>{});
    };
    const bool bias_last = B32 && !perm;
    __syncthreads();  // the observations and the biases are complete in LDS
    init_acc(0, bias_last && !narrow);
    if (narrow) {
        if constexpr (B32) {
            for (int k = 0; k < O; ++k) {
                float xv[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    xv[i] = to_f(*reinterpret_cast<const bf16_t*>(dlds + (32 * i + lr) * pitch0 + (((k >> 3) ^ (lr & 15)) * 16) + (k & 7) * 2));
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint4 w = *reinterpret_cast<const uint4*>(wst + k * 128 + (16 * q + 8 * lg) * 2);
                    const uint32_t wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float wf = __uint_as_float((u & 1) ? wv[u >> 1] & 0xffff0000u : wv[u >> 1] << 16);
#pragma unroll
                        for (int i = 0; i < NI; ++i)
                            acc[i][q >> 1][8 * (q & 1) + u] = __builtin_fmaf(xv[i], wf, acc[i][q >> 1][8 * (q & 1) + u]);
                    }
                }
            }
        }
    } else {
        for (int s = 0; s < n0; ++s) {
            if (s + 1 == n0) {
                const int ol = opaque(lane);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    if constexpr (B32) {
                        w0[b] &= keep[b & 1];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) w0[b][e] = kept(ol, b, e) > 0 ? w0[b][e] : 0u;
                    }
                }
            }
            products(w0, s, pitch0);
            if (s + 1 < n0) load_w(w0, Wp + (s + 1) * 128, O, KS);
        }
    }
    if (!EARLY) fill();
    finish_layer(0, bias_last && !narrow);
    for (int l = 1; l < L; ++l) {
        __syncthreads();  // the layer's input is complete in LDS
        init_acc(l, bias_last);
        for (int s = 0; s < S1; s += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                products(wf[u], s + u, PITCH);
                __builtin_amdgcn_sched_barrier(0);
                fetch(wf[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        finish_layer(l, bias_last);
    }
    // output layer: a wave takes 16 rows at a time; lane (ln, kg) supplies row ln / output ln at contraction chunk
    // 4 u + kg and receives output ln of rows 4 kg + e.  What it reads from memory (the first batch of weights, biases, log
    // sigmas, the rows' noise) is requested together and ahead of the barrier: behind it, where each was needed, it was four
    // round trips one after the other (a step of 32 preferences x 256 rows of 3 x 256: 14.9 us a network, 14.3 now).
    const int ln = lane & 15, kg = lane >> 4;
    constexpr int NU = WP / VE / 4;             // contraction steps
    constexpr int NB = NU % 8 == 0 ? 8 : NU % 6 == 0 ? 6 : NU;  // steps whose operands are requested together
    const bool b_ok = ln < net.out_dim, a_ok = ln < net.adim;   // lanes that hold an output, an action mean
    const int oc = b_ok ? ln : net.out_dim - 1;
    const char* wr = Wp + (net.head_mat_off + (int64_t)oc * W) * ES;
    auto load_fb = [&](u32x4_t (&fb)[NB], int b0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int ch = 4 * (b0 + u) + kg;
            fb[u] = *reinterpret_cast<const u32x4_t*>(wr + (ch * VE < W ? ch : 0) * 16);
        }
    };
    uint32_t orow[4];  // (rows of a time-major tensor stay below 2^31)
    float noise[4];
    auto load_rows = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + 16 * i + 4 * kg + e;
            orow[e] = (uint32_t)net.rm.row(p, m < net.M ? m : net.M - 1);
            noise[e] = 0.f;
            if (net.eps && a_ok && m < net.M) noise[e] = net.eps[(int64_t)orow[e] * net.adim + ln];
        }
    };
    u32x4_t fb[NB];
    float hb = 0.f, ls_p = 0.f;
    if (wave < RT) {
        load_fb(fb, 0);
        hb = bp[net.head_vec_off + oc];
        if (net.eps && a_ok && !net.sig_state) ls_p = bp[net.logsig_off + ln];
        load_rows(wave);
    }
    __syncthreads();
    for (int i = wave; i < RT; i += NW) {
        const unsigned char* hrow = dlds + (16 * i + ln) * PITCH;
        float4_t c = {0.f, 0.f, 0.f, 0.f}, c2 = {0.f, 0.f, 0.f, 0.f};
        if (i != wave) {
            load_fb(fb, 0);
            load_rows(i);
        }
#pragma unroll
        for (int b0 = 0; b0 < NU; b0 += NB) {
            if (b0 > 0) load_fb(fb, b0);
            uint4 fa[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) fa[u] = *reinterpret_cast<const uint4*>(hrow + (((4 * (b0 + u) + kg) ^ ln) * 16));
            if constexpr (!WHOLE) {  // zero beyond W, as h is
#pragma unroll
                for (int u = 0; u < NB; ++u)
                    if ((4 * (b0 + u) + kg) * VE >= W) fb[u] = u32x4_t{0, 0, 0, 0};
            }
#pragma unroll
            for (int u = 0; u < NB; u += 2) {
                Mma16<T>::run(fa[u], __builtin_bit_cast(uint4, fb[u]), c);
                Mma16<T>::run(fa[u + 1], __builtin_bit_cast(uint4, fb[u + 1]), c2);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] += c2[e];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + 16 * i + 4 * kg + e;
            const bool ok = m < net.M && b_ok;
            const float z = c[e] + hb;
            const float o = (ln < net.tanh_cols) ? tanhf(z) : z;
            const int64_t row = orow[e];
            float term = 0.f;
            // a state-dependent log sigma sits adim columns to the right, in the same group of 16 lanes
            const float ls_s = __shfl(o, (lane & 48) | ((ln + net.adim) & 15), 64);
            if (ok) {
                net.out[row * net.out_dim + ln] = o;
                if (SAVE) net.saved_out[((int64_t)p * net.M + m) * OUT_PITCH + ln] = o;
                if (net.eps && a_ok) {
                    const float ls = net.sig_state ? ls_s : ls_p;
                    const float ep = noise[e];
                    net.act[row * net.adim + ln] = o + expf(ls) * ep;
                    term = -0.5f * ep * ep - ls;
                }
            }
            if (net.eps) {
                term += __shfl_xor(term, 8, 64);
                term += __shfl_xor(term, 4, 64);
                term += __shfl_xor(term, 2, 64);
                term += __shfl_xor(term, 1, 64);
                if (m < net.M && ln == 0) net.logp[row] = term - 0.918938533204672742f * (float)net.adim;
            }
        }
    }
}

// ---- host side: one launch function per (type, SAVE), each instantiated in a translation unit of its own ----------
template <typename T, bool SAVE, int NW, int RT, bool WHOLE>
static void fwd_launch_w(const FwdArgs& a, int n_tiles, hipStream_t s) {
    const int lds = fwd_lds_bytes(sizeof(T), a.O, a.W, a.L, RT);
    static std::atomic<uint64_t> allowed{0};  // devices on which the kernel may take more LDS than the default (a bit each)
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (!(allowed.load(std::memory_order_relaxed) & bit)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_fwd<T, SAVE, NW, RT, WHOLE>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        allowed.fetch_or(bit, std::memory_order_relaxed);
    }
    k_mlp_fwd<T, SAVE, NW, RT, WHOLE><<<n_tiles, 64 * NW, lds, s>>>(a);
}
template <typename T, bool SAVE, int NW, int RT>
static void fwd_launch(const FwdArgs& a, int n_tiles, hipStream_t s) {
    if (a.W == 64 * NW) fwd_launch_w<T, SAVE, NW, RT, true>(a, n_tiles, s);
    else fwd_launch_w<T, SAVE, NW, RT, false>(a, n_tiles, s);
}
template <typename T, bool SAVE, int NW>
static void fwd_launch_rt(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    constexpr int LOW = fwd_low(sizeof(T));
    if constexpr (fwd_has_high(sizeof(T), NW)) {
        if (fwd_compiled(sizeof(T), NW, rt) == 2 * LOW) { fwd_launch<T, SAVE, NW, 2 * LOW>(a, n_tiles, s); return; }
    }
    fwd_launch<T, SAVE, NW, LOW>(a, n_tiles, s);
}
template <typename T, bool SAVE>
static void fwd_launch_all(const FwdArgs& a, int rt, int n_tiles, hipStream_t s) {
    switch (fwd_waves(a.W)) {
        case 1: fwd_launch_rt<T, SAVE, 1>(a, rt, n_tiles, s); break;
        case 2: fwd_launch_rt<T, SAVE, 2>(a, rt, n_tiles, s); break;
        case 3: fwd_launch_rt<T, SAVE, 3>(a, rt, n_tiles, s); break;
        case 4: fwd_launch_rt<T, SAVE, 4>(a, rt, n_tiles, s); break;
        case 6: fwd_launch_rt<T, SAVE, 6>(a, rt, n_tiles, s); break;
        default: fwd_launch_rt<T, SAVE, 8>(a, rt, n_tiles, s); break;
    }
}
