// Fused target-network forward of fp32 networks of width 256 and less (paper Sec. III-C, rollout and update phases): the
// whole network in one launch, its products on the bf16 matrix instructions (split3: every operand the exact sum of three bf16
// values, six products of parts).
//
// A workgroup of NW waves carries ROWS = 32 RB rows of one preference through every layer.  The activations of the tile live in
// LDS as three planes of bf16 parts, split once, in the epilogue that makes them; wave w owns output features [32 w, 32 w + 32)
// for all rows, so its slice of W_l(p) is used by no other wave.  W travels a super-step (a 128-byte line of each of the 32 rows,
// 4 KB) at a time: requested into registers D super-steps ahead, across layer ends, through 4 KB of LDS of the wave's own into
// fragment order one super-step ahead, and split there: some 100 vector instructions beside 12 RB products of 32 cycles.
// What bounds it: one tile runs on a CU, so its ends and epilogues leave the matrix pipe idle.  16 preferences x 8192 rows of 3 x
// 256: the pipe is busy 0.39 of the time (0.33 saving) at 1.95 GHz; of 61 to 67 thousand cycles of a tile of 64 rows each hidden
// layer's products take 12.5 to 17.6 (12.3 of the pipe's), its epilogue with the barriers 4.8 to 9.8, observations and first layer 7 to 8,
// the output layer up to 9.  us plain / saving: 374 / 430 on the fp32 instructions, 268 / 341 so.  (64 features a wave, four waves: 306;
// fragments and the split of W another half super-step ahead: no change; the waves of a SIMD at two priorities: none.)
#pragma once

#include "fused_fwd.h"

// what a row's 16-byte chunks are XORed with: the sixteen rows that a 16-byte read serves at a time fall into different banks
__device__ inline int split_swz(int row, int pitch) {
    return pitch == 64 ? (row >> 2) & 3 : (pitch & 128) ? (row >> 1) & 7 : row & 15;
}
// super-steps requested ahead (a divisor of those of a hidden layer)
constexpr int split_depth(int s1, int rb) { return (s1 == 5 || s1 == 3) && rb == 1 ? s1 : s1 % 2 == 0 ? 2 : 1; }

template <bool SAVE, int NW, int RB, bool WHOLE>
__global__ __launch_bounds__(64 * NW, 2) void k_mlp_fwd_split(FwdArgs a) {
    constexpr int WP = 32 * NW, ROWS = 32 * RB, S1 = NW, PITCH = split_pitch(WP);
    constexpr int D = split_depth(S1, RB);
    static_assert(S1 % D == 0, "the ring of requests wraps at layer ends");
    extern __shared__ __align__(16) unsigned char dlds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const FwdNet& net = a.net;
    const int p = tile / net.tiles_m, m0 = (tile % net.tiles_m) * ROWS;
    const int O = a.O, W = WHOLE ? WP : a.W, L = a.L;
    const float* Wp = reinterpret_cast<const float*>(net.theta_mat) + (int64_t)p * net.mat_len;
    const float* bp = net.theta_vec + (int64_t)p * net.vec_len;
    const int n0 = (O + 31) / 32;  // super-steps of the first layer
    const int pitch0 = split_pitch(O);
    const int plane = ROWS * (pitch0 > PITCH ? pitch0 : PITCH);
    unsigned char* wst = dlds + 3 * plane + wave * 4096;  // this wave's super-step of W; in an epilogue, its store patch
    float* sbias = reinterpret_cast<float*>(dlds + 3 * plane + NW * 4096);  // [L][WP]
    const int lr = lane & 31, lg = lane >> 5;
    const int wrow = swap_bits23(lr);  // W rows in an order that gives a lane eight consecutive features

    // W in LDS: 32 feature rows of eight 16-byte chunks, chunk c of row R at position c ^ ((R >> 1) & 7).  Request b of lane l is
    // position l & 7 of row 8 b + (l >> 3).  Features beyond W repeat the last row (zeroed in the epilogue).  A request past the
    // end of a row meets zero activations; what it finds in another row may only be infinite or undefined, and then the block
    // is multiplied again.
    auto load_w = [&](u32x4_t (&w)[4], const float* base, int ld) __attribute__((always_inline)) {
        const int ol = opaque(lane);  // (formed here: addresses held across the products would cost them registers)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int row = 8 * b + (ol >> 3), f = 32 * wave + row;
            const uint32_t at = (uint32_t)((WHOLE || f < W ? f : W - 1) * ld) * 4u + (uint32_t)(((ol & 7) ^ ((row >> 1) & 7)) * 16);
            w[b] = *reinterpret_cast<const chunk2_t*>(reinterpret_cast<const char*>(base) + at);
        }
    };
    u32x4_t raw[2][2];  // the lane's eight values of the two products of a super-step
    auto stage = [&](const u32x4_t (&w)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b) *reinterpret_cast<u32x4_t*>(wst + b * 1024 + lane * 16) = w[b];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                raw[kk][h] = *reinterpret_cast<const u32x4_t*>(wst + wrow * 128 + (((4 * kk + 2 * lg + h) ^ ((wrow >> 1) & 7)) * 16));
    };
    u32x4_t w0[4];
    // requests of the hidden layers; past the last layer the cursor repeats a valid one, so that every super-step has
    // the same number of loads in flight
    u32x4_t wf[D][4];
    int cl = 1, cs = 0;
    auto fetch = [&](u32x4_t (&w)[4]) __attribute__((always_inline)) {
        load_w(w, Wp + (int64_t)W * O + (int64_t)(cl - 1) * W * W + cs * 32, W);
        if (++cs == S1) {
            cs = 0;
            cl = cl + 1 < L ? cl + 1 : cl;
        }
    };

    // What the tile starts from is requested together, what is needed first ahead of the rest: observations, biases (a register
    // load later on would stand behind the ring's requests), W_0, the ring.  us, piece by piece and so: 10 preferences x 1850 rows of
    // 2 x 160 with 100 observations, saving, 44.3 and 40.0; 24 x 1000 of 3 x 256 with 120 72.9 and 67.6, saving 84.9 and 80.9.
    {
        constexpr int NT = 64 * NW, NB = 4;  // layers whose biases come along
        constexpr int G = 8 * RB >= 5 * NW ? 5 : (8 * RB + NW - 1) / NW;  // pieces a thread requests together: 128 observations
        // 2^sh pieces of eight values a row, those behind the last super-step skipped, those behind the observations zero
        const int np = 4 * n0, nc = (O + 7) / 8, sh = 32 - __builtin_clz(np - 1), n_id = ROWS << sh;
        const int mlim = SAVE ? a.Mp - m0 : 0;
        const int bf = (int)threadIdx.x < W ? threadIdx.x : W - 1;
        static_assert(NT >= WP, "a bias a thread and layer");
        // the observations, zero-filled to whole steps; rows past the end repeat the last row (their outputs are never stored)
        auto obs_row = [&](int r) __attribute__((always_inline)) {
            return a.x + (uint32_t)net.rm.row(p, m0 + r < net.M ? m0 + r : net.M - 1) * (uint32_t)O;  // (the tensor stays below 4 GiB)
        };
        auto load_x = [&](u32x4_t (&v)[G][2], int first) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = first + g * NT + (int)threadIdx.x, id = i < n_id ? i : n_id - 1;
                obs_get(v[g], obs_row(id >> sh), id & ((1 << sh) - 1), O);
            }
        };
        auto put_piece = [&](const float (&v)[8], int r, int c) __attribute__((always_inline)) {
            uint4 part[3];
            split3<true>(v, part);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<uint4*>(dlds + q * plane + r * pitch0 + ((c ^ split_swz(r, pitch0)) * 16)) = part[q];
            if (SAVE && net.x0 && r < mlim && c < nc)
                store8(reinterpret_cast<float*>(net.x0) + ((int64_t)p * a.Mp + m0 + r) * a.ldx + 8 * c, v);
        };
        auto put_x = [&](u32x4_t (&v)[G][2], int first) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int id = first + g * NT + (int)threadIdx.x, r = id >> sh, c = id & ((1 << sh) - 1);
                float w[8];
                obs_place(w, v[g], c, O);
                if (id < n_id && c < np) put_piece(w, r, c);
            }
        };
        u32x4_t v[G][2];
        int first = 0;
        if (O >= 8) {
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
        load_w(w0, Wp, O);
        if (L > 1) {
#pragma unroll
            for (int u = 0; u < D; ++u) fetch(wf[u]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if ((int)threadIdx.x < WP) {
#pragma unroll
            for (int l = 0; l < NB; ++l)
                if (l < L) sbias[l * WP + threadIdx.x] = bv[l];
            for (int l = NB; l < L; ++l) sbias[l * WP + threadIdx.x] = bp[l * W + bf];
        }
        if (O >= 8) {
            put_x(v, first);
        } else {  // rows shorter than a piece, element by element
            for (int r = threadIdx.x; r < ROWS; r += NT) {
                const float* row = obs_row(r);
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = e < O ? row[e < O ? e : O - 1] : 0.f;
                put_piece(w, r, 0);
                for (int c = 1; c < np; ++c) {
                    const float zero[8] = {};
                    put_piece(zero, r, c);
                }
            }
        }
    }

    // accumulators: 32-row block i: lane (lr, lg) holds row 32 i + lr, features 16 h + 8 lg + u in element 8 h + u
    float16_t acc[RB], low[RB];
    auto init_acc = [&](int l) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4* b = reinterpret_cast<const float4*>(sbias + l * WP + 32 * wave + 16 * h + 8 * lg);
            const float4 b0 = b[0], b1 = b[1];
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                acc[i][8 * h] = b0.x; acc[i][8 * h + 1] = b0.y; acc[i][8 * h + 2] = b0.z; acc[i][8 * h + 3] = b0.w;
                acc[i][8 * h + 4] = b1.x; acc[i][8 * h + 5] = b1.y; acc[i][8 * h + 6] = b1.z; acc[i][8 * h + 7] = b1.w;
            }
        }
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) low[i][e] = 0.f;
    };
    auto split_raw = [&](uint4 (&w)[2][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(raw[kk][e >> 2][e & 3]);
            split3(v, w[kk]);
        }
    };
    auto products = [&](const uint4 (&w)[2][3], int s, int pitch) __attribute__((always_inline)) {
        const unsigned char* as = dlds + lr * pitch;
        const int x = split_swz(lr, pitch);  // (of row 32 i + lr as well)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            uint4 fa[RB][3];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int i = 0; i < RB; ++i)
                    fa[i][q] = *reinterpret_cast<const uint4*>(as + q * plane + i * 32 * pitch + (((4 * s + 2 * kk + lg) ^ x) * 16));
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int i = 0; i < RB; ++i) split_mma(t, w[kk], fa[i], acc[i], low[i]);
        }
    };
    // a value of the tile, from its parts (an infinite one's second part is infinite, its third undefined)
    auto tile_value = [&](int row, int k, int pitch) __attribute__((always_inline)) {
        const unsigned char* at = dlds + row * pitch + (((k >> 3) ^ split_swz(row, pitch)) * 16) + (k & 7) * 2;
        const float v0 = to_f(*reinterpret_cast<const bf16_t*>(at)), v1 = to_f(*reinterpret_cast<const bf16_t*>(at + plane)),
                    v2 = to_f(*reinterpret_cast<const bf16_t*>(at + 2 * plane));
        return __builtin_isinf(v1) ? v1 : v0 + (v1 + v2);
    };
    // the sums of a layer whose input is d_in wide; undefined and infinite ones once more on the fp32 instructions
    auto finish_sums = [&](int l, const float* Wl, int d_in, int pitch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            acc[i] += low[i];
            if (any_undefined(acc[i])) {
                const int f = 32 * wave + wrow;
                const float* wr = Wl + (int64_t)(f < W ? f : W - 1) * d_in;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][e] = sbias[l * WP + 32 * wave + 16 * (e >> 3) + 8 * lg + (e & 7)];
#pragma unroll 1
                for (int k = 0; k < d_in; k += 2) {
                    const int kk = k + lg;
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(kk < d_in ? wr[kk] : 0.f, kk < d_in ? tile_value(32 * i + lr, kk, pitch) : 0.f,
                                                                  acc[i], 0, 0, 0);
                }
            }
        }
    };
    auto epilogue = [&](int l, auto act_tag) __attribute__((always_inline)) {
        constexpr int MODE = decltype(act_tag)::value;
        const int mlim = SAVE ? a.Mp - m0 : 0;
        const int el = opaque(lane), er = el & 31, eg = el >> 5;
        const int64_t at = (int64_t)l * a.lstride + ((int64_t)p * a.Mp + m0) * a.ldh * 4;
        char* Hl = SAVE ? net.H + at : nullptr;
        char* Gl = SAVE ? net.G + at : nullptr;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int row = 32 * i + er;
            __builtin_amdgcn_sched_barrier(0);  // one row block's temporaries at a time
            float g[2][8], v[2][8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int f = 32 * wave + 16 * h + 8 * eg;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    fwd_act<float, MODE>(acc[i][8 * h + u], v[h][u], g[h][u]);
                    if (!WHOLE && f >= W) v[h][u] = g[h][u] = 0.f;
                }
                uint4 part[3];
                split3<MODE != kActTanh>(v[h], part);  // (SiLU's may be as large as its argument)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint4*>(dlds + q * plane + row * PITCH + (((f >> 3) ^ split_swz(row, PITCH)) * 16)) = part[q];
            }
            if (SAVE) {  // through the wave's room for W, so that a store instruction writes whole 128-byte row segments
#pragma unroll
                for (int arr = 0; arr < 2; ++arr) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            *reinterpret_cast<uint4*>(wst + er * 128 + (((4 * h + 2 * eg + b) ^ ((er >> 1) & 7)) * 16)) =
                                pack_chunk<float>((arr ? v[h] : g[h]) + 4 * b);
                    __builtin_amdgcn_wave_barrier();
                    char* dst = arr ? Hl : Gl;
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const int prow = it * 8 + (el >> 3), pc = el & 7, f = 32 * wave + pc * 4;
                        const uint4 u = *reinterpret_cast<const uint4*>(wst + prow * 128 + ((pc ^ ((prow >> 1) & 7)) * 16));
                        if (32 * i + prow < mlim && (WHOLE || f < a.ldh))
                            *reinterpret_cast<uint4*>(dst + (uint32_t)((32 * i + prow) * a.ldh + f) * 4) = u;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    };
    auto finish_layer = [&](int l) __attribute__((always_inline)) {
        __syncthreads();  // every wave has read the layer's input for the last time
        if (a.act == 0) epilogue(l, std::integral_constant<int, kActTanh>{});
        else epilogue(l, std::integral_constant<int, kActSiluPlain>{});
    };
    __syncthreads();  // the observations and the biases are complete in LDS
    init_acc(0);
    for (int s = 0; s < n0; ++s) {
        uint4 w[2][3];
        stage(w0);
        if (s + 1 < n0) load_w(w0, Wp + (s + 1) * 32, O);
        split_raw(w);
        products(w, s, pitch0);
    }
    finish_sums(0, Wp, O, pitch0);
    if (L > 1) {
        stage(wf[0]);
        fetch(wf[0]);
    }
    finish_layer(0);
    for (int l = 1; l < L; ++l) {
        __syncthreads();  // the layer's input is complete in LDS
        init_acc(l);
        for (int s = 0; s < S1; s += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                uint4 w[2][3];
                split_raw(w);
                stage(wf[(u + 1) % D]);
                fetch(wf[(u + 1) % D]);
                products(w, s + u, PITCH);
            }
        }
        finish_sums(l, Wp + (int64_t)W * O + (int64_t)(l - 1) * W * W, W, PITCH);
        finish_layer(l);
    }
    // output layer: a wave takes 16 rows at a time; lane (ln, kg) supplies row ln / output ln at contraction indices
    // 32 u + 8 kg .. + 7 and receives output ln of rows 4 kg + e.  What it reads from memory is requested together and ahead of
    // the barrier.
    const int ln = lane & 15, kg = lane >> 4;
    const bool b_ok = ln < net.out_dim, a_ok = ln < net.adim;  // lanes that hold an output, an action mean
    const int oc = b_ok ? ln : net.out_dim - 1;
    const float* wr = Wp + net.head_mat_off + (int64_t)oc * W;
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
    u32x4_t fb[S1][2];
    float hb = 0.f, ls_p = 0.f;
    if (wave < 2 * RB) {
#pragma unroll
        for (int u = 0; u < S1; ++u) {
            const int k = 32 * u + 8 * kg;
#pragma unroll
            for (int h = 0; h < 2; ++h) fb[u][h] = *reinterpret_cast<const u32x4_t*>(wr + (WHOLE || k < W ? k : 0) + 4 * h);
        }
        hb = bp[net.head_vec_off + oc];
        if (net.eps && a_ok && !net.sig_state) ls_p = bp[net.logsig_off + ln];
        load_rows(wave);
    }
    __syncthreads();
    for (int i = wave; i < 2 * RB; i += NW) {
        float4_t c = {0.f, 0.f, 0.f, 0.f}, c2 = {0.f, 0.f, 0.f, 0.f};
        if (i != wave) load_rows(i);
#pragma unroll
        for (int u = 0; u < S1; ++u) {
            const int k = 32 * u + 8 * kg;
            const bool in = WHOLE || k < W;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = in ? __uint_as_float(fb[u][e >> 2][e & 3]) : 0.f;  // (zero beyond W, as h is)
            uint4 w[3], fa[3];
            split3(v, w);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                fa[q] = *reinterpret_cast<const uint4*>(dlds + q * plane + (16 * i + ln) * PITCH + (((4 * u + kg) ^ split_swz(16 * i + ln, PITCH)) * 16));
            Mma16<bf16_t>::run(fa[0], w[2], c2);
            Mma16<bf16_t>::run(fa[2], w[0], c2);
            Mma16<bf16_t>::run(fa[1], w[1], c2);
            Mma16<bf16_t>::run(fa[0], w[1], c2);
            Mma16<bf16_t>::run(fa[1], w[0], c2);
            Mma16<bf16_t>::run(fa[0], w[0], c);
        }
        c += c2;
        {
            const float t = (c[0] + c[1]) + (c[2] + c[3]);
            if (any_undefined(t)) {  // as in the hidden layers
                c = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int k = 0; k < W; k += 4)
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(tile_value(16 * i + ln, k + kg, PITCH), wr[k + kg], c, 0, 0, 0);
            }
        }
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

// ---- host side -----------------------------------------------------------------------------------------------------
template <bool SAVE, int NW, int RB, bool WHOLE>
static void split_launch_w(const FwdArgs& a, int n_tiles, hipStream_t s) {
    static std::atomic<uint64_t> allowed{0};  // devices on which the kernel may take more LDS than the default (a bit each)
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (!(allowed.load(std::memory_order_relaxed) & bit)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_fwd_split<SAVE, NW, RB, WHOLE>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        allowed.fetch_or(bit, std::memory_order_relaxed);
    }
    k_mlp_fwd_split<SAVE, NW, RB, WHOLE><<<n_tiles, 64 * NW, split_lds_bytes(a.O, a.W, a.L, RB), s>>>(a);
}
template <bool SAVE, int NW, bool WHOLE>
static void split_launch_rb(const FwdArgs& a, int rb, int n_tiles, hipStream_t s) {
    if constexpr (split_most(NW) >= 3) {
        if (rb == 3) { split_launch_w<SAVE, NW, 3, WHOLE>(a, n_tiles, s); return; }
    }
    if constexpr (split_most(NW) >= 2) {
        if (rb == 2) { split_launch_w<SAVE, NW, 2, WHOLE>(a, n_tiles, s); return; }
    }
    split_launch_w<SAVE, NW, 1, WHOLE>(a, n_tiles, s);
}
template <bool SAVE, int NW>
static void split_launch(const FwdArgs& a, int n_tiles, hipStream_t s) {
    if (a.W == 32 * NW) split_launch_rb<SAVE, NW, true>(a, a.split, n_tiles, s);
    else split_launch_rb<SAVE, NW, false>(a, a.split, n_tiles, s);
}
template <bool SAVE>
static void split_launch_all(const FwdArgs& a, int n_tiles, hipStream_t s) {
    switch (split_waves(a.W)) {
        case 1: split_launch<SAVE, 1>(a, n_tiles, s); break;
        case 2: split_launch<SAVE, 2>(a, n_tiles, s); break;
        case 3: split_launch<SAVE, 3>(a, n_tiles, s); break;
        case 4: split_launch<SAVE, 4>(a, n_tiles, s); break;
        case 5: split_launch<SAVE, 5>(a, n_tiles, s); break;
        case 6: split_launch<SAVE, 6>(a, n_tiles, s); break;
        default: split_launch<SAVE, 8>(a, n_tiles, s); break;
    }
}
