// Hypernetwork forward and backward (paper Sec. III-B: H(w) = M f(w) + b, read as rank-r factors on
// shared base weights; with rank < 0 the strictly affine form, every weight its own row of M, which runs
// entirely through the stacked affine map below).  fp32 arithmetic; theta_mat is rounded to bf16 (nearest even) on store when
// the target networks run in bf16.  Every reduction is fixed-order.
#include "mlp_device.h"
#include "morlax_internal.h"
#include "numeric.h"

#include <atomic>
#include <type_traits>

#define DAB_COLS 128  // columns of dW one block of the fused dA/dB kernel walks
#define DAB_NCT (DAB_COLS / 64)

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct HyperWs {
    float *h1, *f, *fac, *dfac, *df_part, *df, *dz2, *dz1, *vecs, *da_part;
    int n_chunk, n_cs;
};

// 64-row tiles of the stacked affine map per chunk of the df partials: at least four, about a thousand chunks at most
static int df_chunk_tiles(int64_t q_total) {
    const int64_t t = ((q_total + 63) / 64 + 1023) / 1024;
    return t < 4 ? 4 : (int)t;
}

static int cu_count() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, cus = 0;
        n = hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 ? cus : 256;
    }
    return n;
}

static HyperWs hyper_ws_layout(const morlax_ctx* c, void* ws, int64_t* total) {
    const int64_t P = c->d.P, F = c->d.hyper_width;
    const bool affine = c->d.rank < 0;  // no factor vector: the leading stacked rows are theta_mat itself
    int64_t fac = affine ? 0 : (c->net[0].fac_len > c->net[1].fac_len ? c->net[0].fac_len : c->net[1].fac_len);
    HyperWs L;
    float* p = reinterpret_cast<float*>(ws);
    auto take = [&](int64_t n) { float* r = p; p += align_up(n, 64); return r; };
    L.h1 = take(P * F);
    L.f = take(P * F);
    L.df = take(P * F);
    L.dz2 = take(P * F);
    L.dz1 = take(P * F);
    {
        int64_t vl = c->net[0].vec_len > c->net[1].vec_len ? c->net[0].vec_len : c->net[1].vec_len;
        L.vecs = take(P * vl);
    }
    L.fac = take(P * fac);
    L.dfac = take(P * fac);
    L.n_chunk = 0;  // chunks of the df partials
    for (int n = 0; n < 2; ++n) {
        const int64_t nt = (c->aff[n].q_total + 63) / 64, per = df_chunk_tiles(c->aff[n].q_total);
        const int nc = (int)((nt + per - 1) / per);
        L.n_chunk = nc > L.n_chunk ? nc : L.n_chunk;
    }
    L.df_part = take((int64_t)L.n_chunk * P * F);
    {
        int wmax = c->d.width > c->d.obs_dim ? c->d.width : c->d.obs_dim;
        L.n_cs = (wmax + DAB_COLS - 1) / DAB_COLS;
        L.da_part = L.n_cs > 1 ? take((int64_t)L.n_cs * P * fac) : nullptr;
    }
    if (total) *total = (int64_t)((char*)p - (char*)ws);
    return L;
}

int64_t hyper_ws_bytes(const morlax_ctx* c) {
    int64_t t = 0;
    hyper_ws_layout(c, nullptr, &t);
    return align_up(t, 256);
}

// ------------------------------------------------------------------------------------------------
// Trunk f(w): h1 = tanh(Wh1 w + bh1), f = tanh(Wh2 h1 + bh2).
// n values from memory by NT threads, N of a thread requested together (a loop that waits for each before the next is a round trip
// to memory a turn)
template <int N, int NT, class Put>
__device__ inline void take(const float* __restrict__ src, int n, Put put) {
    for (int e0 = threadIdx.x; e0 < n; e0 += N * NT) {
        float v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = src[e0 + u * NT < n ? e0 + u * NT : n - 1];
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (e0 + u * NT < n) put(e0 + u * NT, v[u]);
    }
}
struct Trunk {
    const float* w;  // [P][K]
    float *h1, *f;   // [P][F]
    int32_t K;
    int64_t o_wh1, o_bh1, o_wh2, o_bh2;
    __device__ inline float hidden(const float* __restrict__ hp, int p, int j) const {
        float a = hp[o_bh1 + j];
        for (int k = 0; k < K; ++k) a += hp[o_wh1 + (int64_t)j * K + k] * w[p * K + k];
        return tanhf(a);
    }
    // a workgroup's own copy of the features of all preferences in LDS: sw [F][F + 1], sh and sf [P][F]
    __device__ inline void features(const float* __restrict__ hp, float* sw, float* sh, float* sf, int P, int F, bool keep) const {
        take<4, 256>(hp + o_wh2, F * F, [&](int e, float v) { sw[e / F * (F + 1) + e % F] = v; });
        for (int i = threadIdx.x; i < P * F; i += blockDim.x) {
            const float a = hidden(hp, i / F, i % F);
            sh[i] = a;
            if (keep) h1[i] = a;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < P * F; i += blockDim.x) {
            const int p = i / F, j = i % F;
            float a = hp[o_bh2 + j];
            for (int k = 0; k < F; ++k) a += sw[j * (F + 1) + k] * sh[p * F + k];
            a = tanhf(a);
            sf[i] = a;
            if (keep) f[i] = a;
        }
        __syncthreads();
    }
};
// One block per preference.  (A thread's row of Wh2 requested ahead of h1, each value by itself: 3.2 - 3.6 instead of 3.0 us up to 32
// features, 4.8 - 5.8 instead of 3.1 - 3.7 beyond.)
__global__ __launch_bounds__(64) void k_hyper_trunk(Trunk t, const float* __restrict__ hp, int F) {
    __shared__ float sh[MORLAX_MAX_F];
    const int p = blockIdx.x, j = threadIdx.x;
    if (j < F) {
        const float a = t.hidden(hp, p, j);
        sh[j] = a;
        t.h1[p * F + j] = a;
    }
    __syncthreads();
    if (j < F) {
        float a = hp[t.o_bh2 + j];
        for (int i = 0; i < F; ++i) a += hp[t.o_wh2 + (int64_t)j * F + i] * sh[i];
        t.f[p * F + j] = tanhf(a);
    }
}

// Kernel arguments lie in host memory: the first use of each of their cache lines takes a workgroup about half a microsecond,
// and a use whose place depends on another argument takes its own after that one's.  So what a workgroup looks up by its number
// or its row is computed from arguments at fixed places, all of which are on their way at once.  us a call of hypernet_fwd, with
// tables and searches and requests row by row, and so: 4 preferences of 2 x 32 12.6 and 10.8, 11 of 4 x 512 21.4 and 17.7, 128 106
// and 96.

// Offsets inside hparams of the rows of the stacked affine matrix and of their constants: row q of segment s reads M at m[s] + q F
// and c at c[s] + q.  Segments behind the last one start beyond every row.
struct AffineRows {
    int32_t q_total;
    int32_t q0[MORLAX_MAX_SEG], m[MORLAX_MAX_SEG], c[MORLAX_MAX_SEG];
    __device__ inline void offsets(int F, int q, int32_t& mo, int32_t& co) const {
        mo = m[0];
        co = c[0];
#pragma unroll
        for (int s = 1; s < MORLAX_MAX_SEG; ++s) {
            const bool in = q >= q0[s];
            mo = in ? m[s] : mo;
            co = in ? c[s] : co;
        }
        mo += q * F;
        co += q;
    }
};
static AffineRows affine_rows(const AffineTable& at, int F) {
    AffineRows r;
    r.q_total = at.q_total;
    for (int s = 0; s < MORLAX_MAX_SEG; ++s) {
        const bool in = s < at.n_seg;
        r.q0[s] = in ? at.q0[s] : INT32_MAX;
        r.m[s] = in ? (int32_t)(at.hp_m[s] - (int64_t)at.q0[s] * F) : 0;
        r.c[s] = in ? (int32_t)at.hp_c[s] - at.q0[s] : 0;
    }
    return r;
}

// Where the layers of a network are: the first, the first of the square ones with the distance to the next, the output layer.
// (All offsets inside hparams, theta_mat and the factor vector of a preference stay below 2^31.)
struct LayerPlace { int32_t d_out, d_in, hp_w0, mat, fac_a, fac_b; };
struct LayerRule {
    LayerPlace first, hidden, last;
    int32_t hp_step, mat_step, fac_step, n_hidden;  // hidden layers 1 .. n_hidden - 1 are square
    __device__ inline LayerPlace at(int l) const {
        LayerPlace p = l == 0 ? first : l < n_hidden ? hidden : last;
        const int k = l > 0 && l < n_hidden ? l - 1 : 0;
        p.hp_w0 += k * hp_step;
        p.mat += k * mat_step;
        p.fac_a += k * fac_step;
        p.fac_b += k * fac_step;
        return p;
    }
};
static LayerRule layer_rule(const NetDev& nd) {
    auto place = [&](int l) {
        const LayerDev& L = nd.layer[l];
        return LayerPlace{L.d_out, L.d_in, (int32_t)L.hp_w0, (int32_t)L.mat_off, (int32_t)L.fac_a, (int32_t)L.fac_b};
    };
    const int L = nd.n_layers - 1;
    LayerRule r = {place(0), place(1), place(L), 0, 0, 0, L};  // (one hidden layer: `hidden` is not used)
    if (L > 2) {
        r.hp_step = (int32_t)(nd.layer[2].hp_w0 - nd.layer[1].hp_w0);
        r.mat_step = (int32_t)(nd.layer[2].mat_off - nd.layer[1].mat_off);
        r.fac_step = (int32_t)(nd.layer[2].fac_a - nd.layer[1].fac_a);
    }
    return r;
}
// Items of a kernel that takes n0 of the first layer, nh of every square one, the rest of the output layer: item -> layer, item of it
struct LayerItems {
    int32_t n0, nh;
    RowDiv by_nh;
    __device__ inline int layer(const LayerRule& r, int item, int& rest) const {
        if (item < n0) {
            rest = item;
            return 0;
        }
        const int y = item - n0, q = nh > 0 ? (int)by_nh.quotient((uint32_t)y) : 0, k = q < r.n_hidden - 1 ? q : r.n_hidden - 1;
        rest = y - k * nh;
        return 1 + k;
    }
};
static LayerItems layer_items(int n0, int nh) { return {n0, nh, row_div(nh > 0 ? nh : 1)}; }

struct __attribute__((packed, aligned(4))) Run4 { float v[4]; };  // four consecutive floats at any 4-byte boundary

__device__ inline void put_run4(float* d, const float (&v)[4]) {
    Run4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j] = v[j];
    *reinterpret_cast<Run4*>(d) = r;
}
__device__ inline void put_run4(bf16_t* d, const float (&v)[4]) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef bf16x4 bf16x4_any __attribute__((aligned(2)));
    bf16x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = (bf16_t)v[j];
    *reinterpret_cast<bf16x4_any*>(d) = r;
}

// Stacked affine map out[p, q] = c[q] + sum_j M[q, j] f[p, j] on fp32 MFMA: a workgroup takes 64 rows q, wave w of it the
// preferences 16 (w + 4 i) .. + 15.  The 64 rows of M go through LDS (pitch 4 KS + 1: the fragment reads of 16 lanes, four
// rows apart, and of the four lane groups, neighbouring columns, are free of bank conflicts); lane ln of an accumulator
// j holds row 4 ln + j, so that its four accumulators are four consecutive outputs of a preference and a store
// instruction writes 256-byte runs.  Products are added to c in ascending j, four to an instruction, as the sequence of
// fused multiply-adds of a thread per row would: the same bits.  That form (a thread's row of M from 32 loads a
// 128-byte line apart, f through scalar loads whose latency nothing covered) took 45.9 us for 69 thousand rows x 128
// preferences, of which the 36 MB of results are 7; here 22.2.  14.3 us at 15 thousand x 24, here 5.1.
// TRUNK: every workgroup forms the features f(w) of all preferences itself (in LDS; the first one leaves them and h1 for
// the backward pass), which with few of them costs less than the launch in front that it replaces (rule: trunk_fwd_inside).
template <typename TF, int KS, bool TRUNK>  // TF: type of the leading rows' destination (float factors, or theta_mat: strictly affine form)
__global__ __launch_bounds__(256) void k_hyper_affine(AffineRows at, Trunk tk, const float* __restrict__ hp,
                                                     const float* __restrict__ f, TF* __restrict__ fac,
                                                     float* __restrict__ theta_vec, int P, int F,
                                                     int64_t fac_len, int64_t vec_len) {
    constexpr int K4 = 4 * KS;
    __shared__ float sm[64][K4 + 1];
    __shared__ float sc[64];
    __shared__ int32_t so[64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ln = lane & 15, kg = lane >> 4;
    const int q0 = blockIdx.x * 64, q4 = q0 + 4 * ln;
    float cv = 0.f;
    if (threadIdx.x < 64) {  // (rows past the end repeat the last one; they are not stored)
        int32_t m, c;
        at.offsets(F, q0 + lane < at.q_total ? q0 + lane : at.q_total - 1, m, c);
        so[lane] = m;
        cv = hp[c];
    }
    extern __shared__ float tl[];  // TRUNK: Wh2 [F][F + 1], h1 [P][F], f [P][F]
    const float* fs = f;
    if constexpr (TRUNK) fs = tl + F * (F + 1) + P * F;
    float a[KS];
    auto load_f = [&](int p0) {
        const float* fp = fs + (int64_t)(p0 + ln < P ? p0 + ln : P - 1) * F;
#pragma unroll
        for (int k = 0; k < KS; ++k) a[k] = fp[4 * k + kg < F ? 4 * k + kg : 0];
    };
    if (!TRUNK && 16 * wave < P) load_f(16 * wave);
    __syncthreads();
    {
        float v[K4 / 4];
#pragma unroll
        for (int i = 0; i < K4 / 4; ++i) {
            const int idx = threadIdx.x + 256 * i, k = idx % K4;
            v[i] = hp[so[idx / K4] + (k < F ? k : 0)];
        }
        if constexpr (TRUNK) {
            tk.features(hp, tl, tl + F * (F + 1), tl + F * (F + 1) + P * F, P, F, blockIdx.x == 0);
            if (16 * wave < P) load_f(16 * wave);
        }
#pragma unroll
        for (int i = 0; i < K4 / 4; ++i) {
            const int idx = threadIdx.x + 256 * i, k = idx % K4;
            sm[idx / K4][k] = k < F ? v[i] : 0.f;
        }
        if (threadIdx.x < 64) sc[lane] = cv;
    }
    __syncthreads();
    float b[4][KS];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < KS; ++k) b[j][k] = sm[4 * ln + j][4 * k + kg];
    const bool lead = q4 + 3 < fac_len, vec = q4 >= fac_len && q4 + 3 < at.q_total;
    for (int p0 = 16 * wave; p0 < P; p0 += 64) {
        if (F < K4) {  // (masked here and not where they are requested: nobody waits for them before)
#pragma unroll
            for (int k = 0; k < KS; ++k) a[k] = 4 * k + kg < F ? a[k] : 0.f;
        }
        float4_t acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float c = sc[4 * ln + j];
            acc[j] = float4_t{c, c, c, c};
        }
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[j][k], acc[j], 0, 0, 0);
        if (p0 + 64 < P) load_f(p0 + 64);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t p = p0 + 4 * kg + e;
            if (p >= P) continue;
            const float v[4] = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
            if (lead) {
                put_run4(fac + p * fac_len + q4, v);
            } else if (vec) {
                put_run4(theta_vec + p * vec_len + (q4 - fac_len), v);
            } else {  // the run crosses the end of the leading rows, or of the table
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (q4 + j < fac_len) fac[p * fac_len + q4 + j] = cvt<TF>(v[j]);
                    else if (q4 + j < at.q_total) theta_vec[p * vec_len + (q4 + j - fac_len)] = v[j];
                }
            }
        }
    }
}
// Whether a trunk shares a launch with what is next to it: up to 512 preferences x features (us, apart and together, of few
// rows; a launch on the dependent chain is another 1.5 to 2; forward: 128 2.5 + 4.8 and 6.4, 512 4.5 + 5.5 and 9.0, 768
// 4.1 + 5.1 and 9.5, 1024 4.6 + 5.8 and 12.1; backward: 128 3.4 + 3.3 and 3.6, 320 6.2 + 4.6 and 9.4, 768 5.6 + 4.3 and
// 12.7, 1024 6.1 + 4.5 and 15.8), and there
//   forward, where every workgroup of the affine map repeats it: while those are one round of what the chip holds, four a
//     CU for F <= 32 and two above (hypernet_fwd, together and apart: 16 preferences of F = 32, 661 workgroups 9.1 and 10.3,
//     2249 19.2 and 14.1, 12849 90.9 and 61.0; 4 of F = 64, 446 workgroups 1.1 less together, 661 3.5 more)
//   backward, where one workgroup reads all partials: up to 20 million chunks x (preferences x features)^2 (hypernet_bwd: 16
//     of F = 32, 30 chunks 0.5 less together, 101 0.4 more, 989 160 and 148; 8, 166 chunks 1.1 less, 582 0.6 more; 4, 989
//     chunks 135 and 139)
static bool trunk_fwd_inside(int P, int F, int workgroups) { return P * F <= 512 && workgroups <= (F <= 32 ? 1024 : 512); }
static bool trunk_bwd_inside(int P, int F, int n_chunk) { return P * F <= 512 && (int64_t)n_chunk * (P * F) * (P * F) <= 20 << 20; }
template <typename TF>
static void launch_trunk_affine(const AffineTable& table, const Trunk& tk, const float* hp, TF* fac, float* theta_vec, int P, int F,
                                int64_t fac_len, int64_t vec_len, hipStream_t s) {
    const AffineRows at = affine_rows(table, F);
    const int nb = (at.q_total + 63) / 64;
    auto run = [&](auto ks) {
        constexpr int KS = decltype(ks)::value;
        if (trunk_fwd_inside(P, F, nb)) {
            const int lds = (F * (F + 1) + 2 * P * F) * 4;
            k_hyper_affine<TF, KS, true><<<nb, 256, lds, s>>>(at, tk, hp, tk.f, fac, theta_vec, P, F, fac_len, vec_len);
        } else {
            k_hyper_trunk<<<P, 64, 0, s>>>(tk, hp, F);
            k_hyper_affine<TF, KS, false><<<nb, 256, 0, s>>>(at, tk, hp, tk.f, fac, theta_vec, P, F, fac_len, vec_len);
        }
    };
    // as few contraction steps as the features fill, which are also what is read and staged of M (strictly affine 4 x 512, 4
    // preferences, F = 8: 50 us in eight steps, 25 in two, 31 with a thread per row; F = 20: 60, 39 and 37)
    switch ((F + 3) / 4) {
        case 1: case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        case 8: run(std::integral_constant<int, 8>{}); break;
        case 9: case 10: run(std::integral_constant<int, 10>{}); break;
        case 11: case 12: run(std::integral_constant<int, 12>{}); break;
        default: run(std::integral_constant<int, 16>{}); break;
    }
}

// W_l(p) = W0_l + A_l(p) B_l(p) on fp32 MFMA.  A block makes a 64 (d_out) x 128 (d_in) tile of one layer of one preference,
// wave w its rows 16 w .. 16 w + 15.  Operands come straight from memory (B is shared by the four waves through the vector
// cache): no LDS, no barrier, a wave's requests are all on their way at once.  Lane ln of accumulator j holds column 8 ln +
// j, so that its eight accumulators are eight consecutive weights of a row.  Products add in ascending k, as one
// multiply-add after the other would: the same bits.  On the vector ALU from LDS tiles 12.2 us for 24 preferences of 3 x
// 256, here 8.3, 12.9 and 9.8 for 32; 91.6 for 128 of 4 x 512, the same here: 48 for the stores alone, W0 (twice the
// results' bytes, from the caches) and the factors on top.  (W0 shared by two preferences in registers: 101; a
// preference's tiles on one die: 120.)
// Four waves a SIMD, three for ranks beyond 16, asked for by name: with all rows of a tile requested at once the compiler takes 136
// and 172 registers, one wave less, if it is let.  us a call of hypernet_fwd, let and so: bf16, 128 preferences of 4 x 512, rank 16
// 97.8 and 87.4, 12 89.6 and 80.3, 17 153 and 129, 32 177 and 154; 100 of 2 x 160, rank 16 22.6 and 20.8; fp32, 64 of 3 x 256, rank 24
// 43.9 and 41.3, 16 33.4 and 32.8.
template <typename T, int KS>
__global__ __launch_bounds__(256, KS == 8 ? 3 : 4) void k_hyper_materialize(LayerRule lr, LayerItems tiles, RowDiv by_ti0, RowDiv by_ti, const float* __restrict__ hp,
                                                          const float* __restrict__ fac, T* __restrict__ theta_mat, int r,
                                                          int64_t fac_len, int64_t mat_len) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ln = lane & 15, kg = lane >> 4;
    const int p = blockIdx.y;
    int tl;
    const int l = tiles.layer(lr, blockIdx.x, tl);
    const LayerPlace L = lr.at(l);
    const int ti = (L.d_in + 127) / 128, to = (int)(l == 0 ? by_ti0 : by_ti).quotient((uint32_t)tl);  // tiles along d_in
    const int o0 = to * 64 + 16 * wave, i0 = (tl - to * ti) * 128 + 8 * ln;
    if (o0 >= L.d_out) return;
    const int oa = o0 + ln < L.d_out ? o0 + ln : L.d_out - 1;  // row of A this lane feeds
    const float* fp = fac + (int64_t)p * fac_len;
    T* dst = theta_mat + (int64_t)p * mat_len + L.mat;
    // WHOLE: rows of a multiple of four columns, so that four consecutive ones are either all in the matrix or all beyond it.  (With
    // both kinds of requests in branches of their own, as they are here for other rows, the compiler waits for one row before it
    // requests the next.)
    auto tile = [&](auto whole) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        // the lane's columns i0 .. i0 + 7 of a row; what lies beyond the matrix is not stored
        auto row8 = [&](const float* row, float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = i0 + 4 * h;
                if (WHOLE || i + 4 <= L.d_in) {
                    const Run4 q = *reinterpret_cast<const Run4*>(row + (!WHOLE || i < L.d_in ? i : 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * h + e] = q.v[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * h + e] = i + e < L.d_in ? row[i + e] : 0.f;
                }
            }
        };
        float w0[4][8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int o = o0 + 4 * kg + e;
            row8(hp + L.hp_w0 + (int64_t)(o < L.d_out ? o : L.d_out - 1) * L.d_in, w0[e]);
        }
        float a[KS + 1], b[KS + 1][8];  // (KS = 0, rank 0: W0 alone, there are no factors to read)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + kg, kc = k < r ? k : 0;
            a[s] = fp[L.fac_a + (int64_t)oa * r + kc];
            row8(fp + L.fac_b + (int64_t)kc * L.d_in, b[s]);
        }
        float4_t acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bool in = 4 * s + kg < r;  // (both factors: an infinite one beyond the rank would leave an undefined product)
            a[s] = in ? a[s] : 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], in ? b[s][j] : 0.f, acc[j], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int o = o0 + 4 * kg + e;
            if (o >= L.d_out) continue;
            T* d = dst + (int64_t)o * L.d_in + i0;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = w0[e][j] + acc[j][e];
            if (i0 + 8 <= L.d_in && L.d_in % 8 == 0) {
                store8(d, v);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (i0 + j < L.d_in) d[j] = cvt<T>(v[j]);
            }
        }
    };
    if (L.d_in % 4 == 0) tile(std::true_type{});
    else tile(std::false_type{});
}

static Trunk trunk_of(const morlax_ctx* c, int net, const float* w, const HyperWs& L) {
    const NetDev& nd = c->net[net];
    return {w, L.h1, L.f, c->d.K, nd.hp_wh1, nd.hp_bh1, nd.hp_wh2, nd.hp_bh2};
}
static void run_trunk_and_affine(const morlax_ctx* c, int net, const float* hp, const float* w,
                                 const HyperWs& L, float* theta_vec, hipStream_t s) {
    const NetDev& nd = c->net[net];
    launch_trunk_affine<float>(c->aff[net], trunk_of(c, net, w, L), hp, L.fac, theta_vec, c->d.P, c->d.hyper_width, nd.fac_len,
                               nd.vec_len, s);
}

void launch_hypernet_fwd(const morlax_ctx* c, int net, const float* hparams, const float* w,
                         void* theta_mat, float* theta_vec, void* ws, hipStream_t s) {
    const NetDev& nd = c->net[net];
    HyperWs L = hyper_ws_layout(c, ws, nullptr);
    if (c->d.rank < 0) {
        // strictly affine form (Sec. III-B as written): the stacked map writes theta_mat and theta_vec directly
        const Trunk tk = trunk_of(c, net, w, L);
        if (c->d.wdtype == 1)
            launch_trunk_affine<bf16_t>(c->aff[net], tk, hparams, (bf16_t*)theta_mat, theta_vec, c->d.P, c->d.hyper_width,
                                        nd.fac_len, nd.vec_len, s);
        else
            launch_trunk_affine<float>(c->aff[net], tk, hparams, (float*)theta_mat, theta_vec, c->d.P, c->d.hyper_width,
                                       nd.fac_len, nd.vec_len, s);
        return;
    }
    run_trunk_and_affine(c, net, hparams, w, L, theta_vec, s);
    auto ti = [&](int l) { return (nd.layer[l].d_in + 127) / 128; };
    auto tiles = [&](int l) { return ti(l) * ((nd.layer[l].d_out + 63) / 64); };
    const int n_hidden = nd.n_layers - 1, th = n_hidden > 1 ? tiles(1) : 0;
    const dim3 grid(tiles(0) + (n_hidden - 1) * th + tiles(n_hidden), c->d.P);
    const int r = c->d.rank;
    auto pick = [&](auto type) {
        typedef decltype(type) T;
        T* tm = reinterpret_cast<T*>(theta_mat);
        auto run = [&](auto ks) {
            k_hyper_materialize<T, decltype(ks)::value><<<grid, 256, 0, s>>>(layer_rule(nd), layer_items(tiles(0), th), row_div(ti(0)),
                                                                         row_div(ti(1)), hparams, L.fac, tm, r, nd.fac_len, nd.mat_len);
        };
        if (r == 0) run(std::integral_constant<int, 0>{});
        else if (r <= 8) run(std::integral_constant<int, 2>{});
        else if (r <= 16) run(std::integral_constant<int, 4>{});
        else run(std::integral_constant<int, 8>{});
    };
    if (c->d.wdtype == 1) pick(bf16_t{});
    else pick(float{});
}

// ------------------------------------------------------------------------------------------------
// Backward.

// dW0_l = sum_p dW_l(p): four consecutive elements per thread, p ascending.
__device__ inline void dbase_block(const LayerRule& lr, const LayerItems& elems, int64_t mat_len, const float* __restrict__ dmat,
                                   float* __restrict__ dhp, int P, int blk) {
    const int e = (blk * 256 + (int)threadIdx.x) * 4;
    if (e >= mat_len) return;
    int at;
    const int l = elems.layer(lr, e, at);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* src = dmat + e;
    int p = 0;
    for (; p + 8 <= P; p += 8) {  // eight preferences' loads in flight together
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(src + (int64_t)(p + u) * mat_len);
#pragma unroll
        for (int u = 0; u < 8; ++u) { a.x += v[u].x; a.y += v[u].y; a.z += v[u].z; a.w += v[u].w; }
    }
    for (; p < P; ++p) {
        const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)p * mat_len);
        a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
    }
    float* d = dhp + lr.at(l).hp_w0 + at;
    d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w;
}
struct BaseWork {  // blocks of 256 threads that add up dW0: by themselves or, where there are factors, beside those of k_hyper_dAB
    float* dhp;
    int64_t mat_len;
    LayerItems elems;  // elements of theta_mat
    int32_t n, n_dab;  // base blocks, blocks of dA / dB
    // 0: base blocks behind all others.  Else in rows of eight: base rows a row until there are no more, 2^32 times and rounded down,
    // those in front of a row rounded up (so the first row is one of them, and 2^32 puts all of them first).
    uint64_t share;
};
__global__ __launch_bounds__(256) void k_hyper_base(LayerRule lr, BaseWork bw, const float* __restrict__ dmat, int P) {
    dbase_block(lr, bw.elems, bw.mat_len, dmat, bw.dhp, P, blockIdx.x);
}

// Fused dA / dB on fp32 MFMA, one pass over dW:
//   dA_l(p)[o, k] = sum_i dW_l(p)[o, i] B_l(p)[k, i],   dB_l(p)[k, i] = sum_o A_l(p)[o, k] dW_l(p)[o, i].
// A block owns (p, layer, a run of <= DAB_COLS columns).  It walks the 64 x 64 tiles of dW row block by row
// block: wave w multiplies rows 16 w .. of the tile by B^T (dA, finished after the columns of a row block)
// and A^T by columns 16 w .. of the tile (dB, accumulated over all row blocks in registers).
// dW0, which reads the same matrices, runs in the same launch: it is bound by memory, dA / dB by its products (128 preferences of
// 4 x 512, rank 16: 87 us behind 133 as launches of their own, together 182; 24 of 3 x 256: 5.6 + 18 and 22.4).  While the blocks of
// dA / dB are about as many as the chip holds, four a CU and an eighth of that (the first to go, those of the first layer, are
// short), they come first and dW0 runs beside them; from some 80 preferences on up to 3.5 a CU, because a block of dW0 adds its
// preferences eight at a time, one batch behind the other, and is no longer the shorter one.  With more blocks of dA / dB than that
// dW0's are spread evenly among them, in rows of eight consecutive blocks of one kind, one to a die, or come first where there is no
// more than one a CU.  (Block by block every eighth was dA / dB for 9 preferences of 3 x 768, all of them on one die.)
// us a call of hypernet_bwd, spread block by block, in rows of eight, and with dA / dB first: those 9 101, 72, 63; 4 x 512, 16
// preferences (272 blocks) 62, 72, 54, 48 (816) 101, 107, 88, 64 (1088) 117, 116, 109, 80 (1360) 138, 135, 139, 128 (2176) 196, 194,
// 247; 3 x 1024, 44 (1100) 191, 193, 185, 50 (1250) 210, 214, 233; 3 x 384 with 97 observations, 90 (900) 86, 87, 85, 110 (1100) 96, 97,
// 100; 3 x 256, 128 (896) 62, 62, 62, 160 (1120) 87, 85, 89; rank 32, 4 x 512, 50 (850) 146, 150, 133.  In rows, evenly and dW0 first:
// 3 x 256, 146 preferences (144 blocks of dW0) 79, 76, 400 195, 174; 500 of 3 x 128 (48) 134, 126; 3 x 384, 146 (336) 125, 133, 200 160, 163.
// Both go through the layers in order, all preferences of one before the next: what either reads first the
// other finds in the memory-side cache (128 matrices of 512 x 512 are 134 of its 256 MB).  Preference by preference 183 us for
// the 128, layer by layer 165; 22.5 and 19 for the 24, 25 and 22 for 32 of 3 x 256, rank 8.  (A wave on sixteen rows by itself,
// operands four columns a lane, no barrier: 181 and 19.7.)
template <int RT>
__global__ __launch_bounds__(256) void k_hyper_dAB(LayerRule lr, LayerItems runs, RowDiv by_p, BaseWork bw,
                                                  const float* __restrict__ dmat, const float* __restrict__ fac,
                                                  float* __restrict__ dfac, float* __restrict__ da_part, int r, int P,
                                                  int64_t fac_len) {
    constexpr int AP = 16 * RT + 4;
    __shared__ __align__(16) float sW[64][68];
    __shared__ float sA[64][AP];
    __shared__ float sB[DAB_NCT][16 * RT][68];
    int dab = blockIdx.x, base = dab - bw.n_dab;  // number among the blocks of its kind; base < 0: none of the other kind
    if (bw.share) {
        const int row = blockIdx.x >> 3, rows = (bw.n + 7) >> 3;
        auto in_front = [&](int r) { return min((int)((bw.share * r + 0xffffffffu) >> 32), rows); };
        const int before = in_front(row);  // base rows in front of this one
        const bool is_base = in_front(row + 1) != before;
        base = is_base ? before * 8 + (blockIdx.x & 7) : -1;
        dab = (row - before) * 8 + (blockIdx.x & 7);
        if (is_base ? base >= bw.n : dab >= bw.n_dab) return;
    }
    if (base >= 0) {
        dbase_block(lr, bw.elems, bw.mat_len, dmat, bw.dhp, P, base);
        return;
    }
    const int item = (int)by_p.quotient((uint32_t)dab), p = dab - item * P;
    int cs;
    const LayerPlace L = lr.at(runs.layer(lr, item, cs));
    const int c_lo = cs * DAB_COLS;
    const int c_hi = (L.d_in < c_lo + DAB_COLS) ? L.d_in : (c_lo + DAB_COLS);
    const int nct = (c_hi - c_lo + 63) / 64;
    const int n_cs = (L.d_in + DAB_COLS - 1) / DAB_COLS;
    const float* dW = dmat + (int64_t)p * bw.mat_len + L.mat;
    const float* Ap = fac + (int64_t)p * fac_len + L.fac_a;
    const float* Bp = fac + (int64_t)p * fac_len + L.fac_b;
    float* dAp = (n_cs > 1 ? da_part + ((int64_t)cs * P + p) * fac_len : dfac + (int64_t)p * fac_len) + L.fac_a;
    float* dBp = dfac + (int64_t)p * fac_len + L.fac_b;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ln = lane & 15, kg = lane >> 4;
    const bool vec = (L.d_in % 4 == 0);
    float4_t accB[DAB_NCT][RT];
#pragma unroll
    for (int ct = 0; ct < DAB_NCT; ++ct)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) accB[ct][rt] = float4_t{0.f, 0.f, 0.f, 0.f};
    // The tiles are walked row block by row block; the next tile of dW is fetched into registers while the
    // current one is multiplied out of LDS.
    const int nrb = (L.d_out + 63) / 64, ntile = nrb * nct;
    static_assert(DAB_NCT == 2, "one or two tiles a row block");
    // Nothing is in the way of a thread's requests: what lies outside the tile is asked for at its edge and zeroed when it is put
    // into LDS.  (Every value of a row that is no multiple of four long behind a condition of its own was sixteen round trips a tile:
    // 13 preferences of 2 x 512 with 190 observations 48.2 and 30.7 us, 22 of 3 x 384 with 97 36.7 and 23.9.)
    auto fetch = [&](int tile, u32x4_t (&regs)[4]) __attribute__((always_inline)) {
        typedef u32x4_t word_t __attribute__((aligned(4)));
        const int o0 = (nct == 2 ? tile >> 1 : tile) * 64, i0 = c_lo + (nct == 2 ? tile & 1 : 0) * 64;
        const int row = o0 + (int)threadIdx.x / 16, i = i0 + (int)threadIdx.x % 16 * 4;
        // (a matrix stays far below 2^32 bytes: one base, an offset of 32 bits a lane; 64-bit addresses were 0.1 to 0.4 us a call more)
        const char* base = reinterpret_cast<const char*>(dW);
        if (vec || i0 + 64 <= c_hi) {  // four values of a row are all in the tile or all beyond it
            const uint32_t col = (uint32_t)(i < c_hi ? i : c_hi - 4);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                regs[q] = *reinterpret_cast<const word_t*>(base + ((uint32_t)(row + 16 * q < L.d_out ? row + 16 * q : L.d_out - 1) * (uint32_t)L.d_in + col) * 4u);
            return;
        }
        uint32_t col[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) col[e] = (uint32_t)(i + e < c_hi ? i + e : c_hi - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t at = (uint32_t)(row + 16 * q < L.d_out ? row + 16 * q : L.d_out - 1) * (uint32_t)L.d_in;
#pragma unroll
            for (int e = 0; e < 4; ++e) regs[q][e] = *reinterpret_cast<const uint32_t*>(base + (at + col[e]) * 4u);
        }
    };
    auto put = [&](int o0, int i0, const u32x4_t (&regs)[4]) __attribute__((always_inline)) {
        const int row = threadIdx.x / 16, c4 = threadIdx.x % 16 * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4_t v = regs[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = o0 + row + 16 * q < L.d_out && i0 + c4 + e < c_hi ? v[e] : 0u;
            *reinterpret_cast<u32x4_t*>(&sW[row + 16 * q][c4]) = v;
        }
    };
    // a row block's rows of A(p), requested one row block ahead
    constexpr int APT = 64 * 16 * RT / 256;
    float anx[APT];
    auto fetch_a = [&](int rb) {
#pragma unroll
        for (int q = 0; q < APT; ++q) {
            const int idx = threadIdx.x + 256 * q, row = idx / (16 * RT), k = idx % (16 * RT);
            const int o = rb * 64 + row < L.d_out ? rb * 64 + row : L.d_out - 1;
            anx[q] = Ap[(int64_t)o * r + (k < r ? k : 0)];
        }
    };
    u32x4_t nxt[4];
    fetch(0, nxt);
    fetch_a(0);
    {  // the block's columns of B(p), the same for every row block: requested together (one by one they were eight round trips)
        constexpr int BPT = DAB_NCT * 16 * RT * 64 / 256;
        float b[BPT];
        auto each = [&](auto body) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < BPT; ++q) {
                const int idx = threadIdx.x + 256 * q, ct = idx / (16 * RT * 64), k = (idx / 64) % (16 * RT), cc = idx % 64;
                body(b[q], ct, k, cc, c_lo + ct * 64 + cc);
            }
        };
        each([&](float& v, int, int k, int, int i) { v = Bp[(int64_t)(k < r ? k : 0) * L.d_in + (i < c_hi ? i : c_hi - 1)]; });
        each([&](float& v, int ct, int k, int cc, int i) { sB[ct][k][cc] = k < r && i < c_hi ? v : 0.f; });
    }
    for (int rb = 0; rb < nrb; ++rb) {
        const int o0 = rb * 64;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < APT; ++q) {
            const int idx = threadIdx.x + 256 * q;
            sA[idx / (16 * RT)][idx % (16 * RT)] = o0 + idx / (16 * RT) < L.d_out && idx % (16 * RT) < r ? anx[q] : 0.f;
        }
        if (rb + 1 < nrb) fetch_a(rb + 1);
        float4_t accA[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) accA[rt] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ct = 0; ct < DAB_NCT; ++ct) {
            if (ct < nct) {
                __syncthreads();
                put(o0, c_lo + 64 * ct, nxt);
                if (rb * nct + ct + 1 < ntile) fetch(rb * nct + ct + 1, nxt);
                __syncthreads();
#pragma unroll
                for (int kk = 0; kk < 16; ++kk) {
                    const float a = sW[16 * wave + ln][4 * kk + kg];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        accA[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sB[ct][16 * rt + ln][4 * kk + kg], accA[rt], 0, 0, 0);
                }
#pragma unroll
                for (int kk = 0; kk < 16; ++kk) {
                    const int row = 16 * (kk >> 2) + (kk & 3) + 4 * kg;
                    const float b = sW[row][16 * wave + ln];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        accB[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(sA[row][16 * rt + ln], b, accB[ct][rt], 0, 0, 0);
                }
            }
        }
        // dA tile: lane holds factor index 16 rt + ln of rows o0 + 16 wave + 4 kg + e
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = o0 + 16 * wave + 4 * kg + e, k = 16 * rt + ln;
                if (o < L.d_out && k < r) dAp[(int64_t)o * r + k] = accA[rt][e];
            }
    }
    // dB tiles: lane holds column i of factor rows 16 rt + 4 kg + e
#pragma unroll
    for (int ct = 0; ct < DAB_NCT; ++ct)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = c_lo + ct * 64 + 16 * wave + ln, k = 16 * rt + 4 * kg + e;
                if (ct < nct && i < c_hi && k < r) dBp[(int64_t)k * L.d_in + i] = accB[ct][rt][e];
            }
}

// dA of layers wider than one column run: add the column-run partials in order.  Four elements a thread, one layer to
// blockIdx.z; bound by memory.  (One element a thread over the rows of all factors: 33.3 us for 128 preferences of 4 x 512,
// rank 16, here 12.1; 17.8 and 6.8 for 64.)
__global__ __launch_bounds__(256) void k_hyper_dA_merge(NetDev nd, const float* __restrict__ da_part,
                                                       float* __restrict__ dfac, int r, int P) {
    const int p = blockIdx.y;
    const LayerDev L = nd.layer[blockIdx.z];
    const int n_cs = (L.d_in + DAB_COLS - 1) / DAB_COLS, n = L.d_out * r, i = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (n_cs == 1 || i >= n) return;
    const float* src = da_part + (int64_t)p * nd.fac_len + L.fac_a + i;
    float* dst = dfac + (int64_t)p * nd.fac_len + L.fac_a + i;
    const int64_t stride = (int64_t)P * nd.fac_len;
    if (i + 4 <= n) {
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int cs = 0; cs < n_cs; ++cs) {
            const Run4 u = *reinterpret_cast<const Run4*>(src + cs * stride);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += u.v[k];
        }
        put_run4(dst, v);
        return;
    }
    for (int k = 0; i + k < n; ++k) {
        float v = 0.f;
        for (int cs = 0; cs < n_cs; ++cs) v += src[cs * stride + k];
        dst[k] = v;
    }
}

__device__ inline float grad_row(const float* __restrict__ dfac, const float* __restrict__ dvec, int64_t p, int q,
                                 int64_t fac_len, int64_t vec_len) {
    return (q < fac_len) ? dfac[p * fac_len + q] : dvec[p * vec_len + (q - fac_len)];
}

// From the gradient g of the stacked affine rows (fp32 MFMA, fixed orders):
//   dM[q, :] = sum_p g[p, q] f[p, :],  dc[q] = sum_p g[p, q] (four interleaved shares of the preferences, each in
//   order, added in a fixed order),  part[chunk, p, j] = sum over the chunk's rows q of g[p, q] M[q, j].
// A chunk is tpw tiles of 64 rows.  Workgroups of eight waves have two roles:
//   df: 128 preferences (16 a wave) walk a chunk's tiles in order; the tile of g (a preference's 64 values one 256-byte
//       run) and of M go through LDS, the next ones are in flight in registers meanwhile.  LDS pitches: g 68 floats,
//       M 16 JT + 16 (reads free of conflicts).
//   dM: a wave takes one tile and all preferences, operands straight from memory: lane ln reads four consecutive rows
//       of a preference, so that a request covers 256-byte runs; no LDS, no barrier, nothing carried between tiles.
// FINE (more than DMF_P preferences): every tile is summed by itself and added to those before it.  Sums of 64 rows are
// what such problems had before; one sum over a chunk is less precise (the trunk's gradients against 64 bits, 130 to 512
// preferences, means of eight inputs: 2.6e-7 to 4.9e-7 of their norm in sums of 64 rows, 3.3e-7 to 5.7e-7 in whole chunks,
// 2.6e-7 to 5.1e-7 here).
// Bound by the latency of g, which both roles read.  All df workgroups, the long ones, come first.  Dealt in turn, one to
// every one or three of dM, they met on the same dies, and within a die on the same shader engines; with four waves and 64
// preferences a workgroup, more than 64 preferences read M and walked the tiles twice.  hypernet_bwd (us) with both roles in
// one, so dealt, and here: strictly affine 3 x 512, 32 preferences 158, 197, 89; 4 x 512, 100 preferences 331, 342, 251.
// The kernel at low rank: 69 thousand rows x 128 preferences 59, 39, 32; 15 thousand x 24 35, 11.4, 11.1; 2600 x 4 23, 10.7, 10.2.
#define DMF_Q 64
#define DMF_W 8             // waves of a workgroup
#define DMF_P (16 * DMF_W)  // preferences of a df workgroup
#define DMF_TB 4            // tiles of a short chunk
// SHORT (up to so many preferences, 32 or 64, in chunks of four tiles; 0: any): a df workgroup requests all of its chunk together
// instead of tile by tile, each behind the one before (rule and both sides' times: dm_df_brief); the products are the same, in the
// same order.
template <int JT, bool FINE, int SHORT>
__global__ __launch_bounds__(64 * DMF_W, JT == 2 ? 4 : 2) void k_hyper_dM_df(const float* __restrict__ hp, AffineRows at, const float* __restrict__ f,
                                                    const float* __restrict__ dfac, const float* __restrict__ dvec,
                                                    float* __restrict__ dhp, float* __restrict__ part, int P, int F,
                                                    int64_t fac_len, int64_t vec_len, int n_tiles, int tpw,
                                                    int n_p, int n_df, int dm_t) {
    constexpr int PD = 68, PJ = 16 * JT + 16, TB = SHORT ? DMF_TB : 1, DP = SHORT ? SHORT : DMF_P;
    extern __shared__ __align__(16) float dml[];
    float(*Dl)[PD] = reinterpret_cast<float(*)[PD]>(dml);                 // [TB * DP]
    float(*Ml)[PJ] = reinterpret_cast<float(*)[PJ]>(dml + TB * DP * PD);  // [TB * DMF_Q]
    int32_t* Rl = reinterpret_cast<int32_t*>(dml + TB * (DP * PD + DMF_Q * PJ));  // offsets of rows of M: twice eight tiles and the table of segments, or the chunk's
    const int q_total = at.q_total;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ln = lane & 15, kg = lane >> 4;
    if ((int)blockIdx.x >= n_df) {  // dM and dc of one tile a wave (no barrier: the waves are on their own)
        const int tile = dm_t * xcd_remap(blockIdx.x - n_df, gridDim.x - n_df) + wave;
        if (wave >= dm_t || tile >= n_tiles) return;
        const int q0 = tile * DMF_Q, q4 = q0 + 4 * ln;
        int32_t mo, co;  // of row q0 + lane
        if constexpr (SHORT > 0) {
            at.offsets(F, q0 + lane < q_total ? q0 + lane : q_total - 1, mo, co);
        } else {  // looked up by their segment: not needed before the results are there
            int sg = 0;
#pragma unroll
            for (int s = 1; s < MORLAX_MAX_SEG; ++s) sg = q0 + lane >= at.q0[s] ? s : sg;
            mo = at.m[sg] + (q0 + lane) * F;
            co = at.c[sg] + q0 + lane;
        }
        float4_t acc[4][JT];
        float dc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) acc[mt][jt] = float4_t{0.f, 0.f, 0.f, 0.f};
        // whole: the tile's rows are all leading rows, or all theta_vec rows; the others are read one by one
        auto walk = [&](auto whole) {
            constexpr bool WHOLE = decltype(whole)::value;
            const float* src = q0 < fac_len ? dfac + q4 : dvec + (q4 - fac_len);
            const int64_t stride = q0 < fac_len ? fac_len : vec_len;
            constexpr int U = 4;  // contraction steps whose operands are requested together
            for (int k0 = 0; 4 * k0 < P; k0 += U) {
                Run4 g[U];
                float b[U][JT];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = 4 * (k0 + u) + kg, pc = p < P ? p : P - 1;
                    if constexpr (WHOLE) {
                        g[u] = *reinterpret_cast<const Run4*>(src + pc * stride);
                    } else {
#pragma unroll
                        for (int mt = 0; mt < 4; ++mt)
                            g[u].v[mt] = q4 + mt < q_total ? grad_row(dfac, dvec, pc, q4 + mt, fac_len, vec_len) : 0.f;
                    }
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt) b[u][jt] = f[(int64_t)pc * F + (16 * jt + ln < F ? 16 * jt + ln : 0)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ok = 4 * (k0 + u) + kg < P;
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt) b[u][jt] = ok && 16 * jt + ln < F ? b[u][jt] : 0.f;
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) {
                        const float v = ok ? g[u].v[mt] : 0.f;
                        dc[mt] += v;
#pragma unroll
                        for (int jt = 0; jt < JT; ++jt)
                            acc[mt][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, b[u][jt], acc[mt][jt], 0, 0, 0);
                    }
                }
            }
        };
        if (q0 + DMF_Q <= fac_len || (q0 >= fac_len && q0 + DMF_Q <= q_total)) walk(std::true_type{});
        else walk(std::false_type{});
        // lane holds feature j = 16 jt + ln of rows q0 + 4 (4 kg + e) + mt
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int q = q0 + 16 * kg + 4 * e + mt;
                const int32_t to = __shfl(mo, 16 * kg + 4 * e + mt, 64);
                if (q < q_total) {
                    float* mr = dhp + to;
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt)
                        if (16 * jt + ln < F) mr[16 * jt + ln] = acc[mt][jt][e];
                }
            }
        // dc: lane group kg holds share kg of rows q4 .. q4 + 3
        float mine = 0.f;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            dc[mt] += __shfl_xor(dc[mt], 16, 64);
            dc[mt] += __shfl_xor(dc[mt], 32, 64);
            if (kg == mt) mine = dc[mt];
        }
        const int32_t to = __shfl(co, 4 * ln + kg, 64);
        if (q4 + kg < q_total) dhp[to] = mine;
        return;
    }
    // df partials of preferences p0 .. p0 + 15 (this wave's)
    const int id = xcd_remap(blockIdx.x, n_df), chunk = id / n_p, pb = id % n_p * DMF_P, p0 = pb + 16 * wave;
    const int t_lo = chunk * tpw, t_hi = (t_lo + tpw < n_tiles) ? (t_lo + tpw) : n_tiles;
    constexpr int MPT = DMF_Q * 16 * JT / (64 * DMF_W);
    float4_t accF[JT];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) accF[jt] = float4_t{0.f, 0.f, 0.f, 0.f};
    float4_t sumF[FINE ? JT : 1];  // FINE: the sum of the tiles before this one
    if constexpr (SHORT > 0) {
        float g[TB][DP / DMF_W], m[TB][MPT];
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int i = 0; i < DP / DMF_W; ++i) {
                const int pp = wave + DMF_W * i, q = (t_lo + t) * DMF_Q + lane;
                g[t][i] = grad_row(dfac, dvec, pp < P ? pp : P - 1, q < q_total ? q : q_total - 1, fac_len, vec_len);
            }
        if (threadIdx.x < TB * DMF_Q) {
            const int q = t_lo * DMF_Q + (int)threadIdx.x;
            int32_t mo, co;
            at.offsets(F, q < q_total ? q : q_total - 1, mo, co);
            Rl[threadIdx.x] = mo;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int i = 0; i < MPT; ++i) {
                const int idx = threadIdx.x + 64 * DMF_W * i, qq = idx / (16 * JT), j = idx % (16 * JT);
                m[t][i] = hp[Rl[t * DMF_Q + qq] + (j < F ? j : 0)];
            }
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int i = 0; i < DP / DMF_W; ++i) {
                const int pp = wave + DMF_W * i;
                Dl[t * DP + pp][lane] = pp < P && (t_lo + t) * DMF_Q + lane < q_total ? g[t][i] : 0.f;
            }
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int i = 0; i < MPT; ++i) {
                const int idx = threadIdx.x + 64 * DMF_W * i, qq = idx / (16 * JT), j = idx % (16 * JT);
                Ml[t * DMF_Q + qq][j] = (t_lo + t) * DMF_Q + qq < q_total && j < F ? m[t][i] : 0.f;
            }
        __syncthreads();
        if (p0 >= P) return;
        for (int t = 0; t < t_hi - t_lo; ++t)
#pragma unroll
            for (int kk = 0; kk < DMF_Q / 4; ++kk) {
                const float a = Dl[t * DP + 16 * wave + ln][4 * kk + kg];
#pragma unroll
                for (int jt = 0; jt < JT; ++jt)
                    accF[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Ml[t * DMF_Q + 4 * kk + kg][16 * jt + ln], accF[jt], 0, 0, 0);
            }
    } else {
        float nxt[DMF_P / DMF_W], mnx[MPT];
        static_assert(64 * DMF_W == 8 * DMF_Q, "a thread a row of eight tiles");
        // the offsets of the rows of M of the chunk's `eight`-th eight tiles, from a copy of the table in LDS.  (From the arguments 84
        // scalars lived through the loop, spilled into vector registers: beyond 128 preferences past 128 of them, where a CU holds one
        // workgroup instead of two.  139 preferences of a strictly affine 4 x 512 network 451 us a launch, 343 here.)
        int32_t* tab = Rl + 16 * DMF_Q;
        auto fill_rows = [&](int eight) {
            const int q0 = (t_lo + 8 * eight) * DMF_Q + (int)threadIdx.x, q = q0 < q_total ? q0 : q_total - 1;
            int s = 0;  // the last segment that starts at or before q
#pragma unroll
            for (int step = 16; step > 0; step >>= 1) s = q >= tab[s + step] ? s + step : s;
            Rl[(eight & 1) * 8 * DMF_Q + threadIdx.x] = tab[32 + s] + q * F;
        };
        auto fetch = [&](int tile) {
            const int q = tile * DMF_Q + lane;
#pragma unroll
            for (int i = 0; i < DMF_P / DMF_W; ++i) {
                const int pp = pb + wave + DMF_W * i;
                nxt[i] = (pp < P && q < q_total) ? grad_row(dfac, dvec, pp, q, fac_len, vec_len) : 0.f;
            }
#pragma unroll
            for (int i = 0; i < MPT; ++i) {
                const int idx = threadIdx.x + 64 * DMF_W * i, qq = idx / (16 * JT), j = idx % (16 * JT);
                mnx[i] = (tile * DMF_Q + qq < q_total && j < F) ? hp[Rl[((tile - t_lo) & 15) * DMF_Q + qq] + j] : 0.f;
            }
        };
        if constexpr (FINE) {
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) sumF[jt] = accF[jt];
        }
        static_assert(MORLAX_MAX_SEG <= 32, "five halvings");
        if (threadIdx.x < 32) {
            const int s = threadIdx.x < MORLAX_MAX_SEG ? threadIdx.x : 0;
            tab[threadIdx.x] = threadIdx.x < MORLAX_MAX_SEG ? at.q0[s] : INT32_MAX;
            tab[32 + threadIdx.x] = at.m[s];
        }
        __syncthreads();
        fill_rows(0);
        __syncthreads();
        fetch(t_lo);
        for (int tile = t_lo; tile < t_hi; ++tile) {
            __syncthreads();  // the previous tile's readers are done
#pragma unroll
            for (int i = 0; i < DMF_P / DMF_W; ++i) Dl[wave + DMF_W * i][lane] = nxt[i];
#pragma unroll
            for (int i = 0; i < MPT; ++i) {
                const int idx = threadIdx.x + 64 * DMF_W * i;
                Ml[idx / (16 * JT)][idx % (16 * JT)] = mnx[i];
            }
            if (((tile - t_lo) & 7) == 6) fill_rows(((tile - t_lo) >> 3) + 1);  // (before the tile behind the next asks for them)
            __syncthreads();
            if (tile + 1 < t_hi) {
                fetch(tile + 1);
            }
            if (p0 < P) {
#pragma unroll
                for (int kk = 0; kk < DMF_Q / 4; ++kk) {
                    const float a = Dl[16 * wave + ln][4 * kk + kg];
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt)
                        accF[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Ml[4 * kk + kg][16 * jt + ln], accF[jt], 0, 0, 0);
                }
            }
            if constexpr (FINE) {
#pragma unroll
                for (int jt = 0; jt < JT; ++jt) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sumF[jt][e] += accF[jt][e];
                    accF[jt] = float4_t{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
    }
    // lane holds feature j = 16 jt + ln of preferences p0 + 4 kg + e
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pp = p0 + 4 * kg + e, j = 16 * jt + ln;
            if (pp < P && j < F) part[((int64_t)chunk * P + pp) * F + j] = FINE ? sumF[FINE ? jt : 0][e] : accF[jt][e];
        }
}

// Trunk backward, stage 1: df[p, j] = sum_chunk part; dz2 = df * (1 - f^2); dz1 = (dz2 Wh2) * (1 - h1^2).  A block
// takes the 64 / F preferences that fit into 64 outputs, so that dz1 follows out of LDS in the launch that made dz2;
// the four thread groups take the chunks c = g, g + 4, ... and are merged in group order.  Bound by latency (a few
// hundred KB): what counts is launches and dependent round trips.
__global__ __launch_bounds__(256) void k_hyper_trunk_bwd_a(const float* __restrict__ hp, const float* __restrict__ part,
                                                          int n_chunk, const float* __restrict__ f,
                                                          const float* __restrict__ h1, float* __restrict__ dz2,
                                                          float* __restrict__ dz1, int P, int F, int64_t o_wh2) {
    __shared__ float red[4][64];
    __shared__ float z2[64];
    __shared__ float wh2[MORLAX_MAX_F * MORLAX_MAX_F];
    const int o = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int PF = P * F, per = (64 / F) * F;
    const int i = blockIdx.x * per + o;
    const bool live = o < per && i < PF;
    take<4, 256>(hp + o_wh2, F * F, [&](int e, float v) { wh2[e] = v; });
    float a = 0.f;
    if (live) {
        int c = g;
        for (; c + 60 < n_chunk; c += 64) {  // sixteen chunks of this group per batch, loads in flight together
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)(c + 4 * u) * PF + i];
#pragma unroll
            for (int u = 0; u < 16; ++u) a += v[u];
        }
        for (; c + 12 < n_chunk; c += 16) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = part[(int64_t)(c + 4 * u) * PF + i];
#pragma unroll
            for (int u = 0; u < 4; ++u) a += v[u];
        }
        for (; c < n_chunk; c += 4) a += part[(int64_t)c * PF + i];
    }
    red[g][o] = a;
    __syncthreads();
    if (g == 0 && live) {
        const float fv = f[i];
        const float z = (red[0][o] + red[1][o] + red[2][o] + red[3][o]) * (1.f - fv * fv);
        z2[o] = z;
        dz2[i] = z;
    }
    __syncthreads();
    if (g == 0 && live) {
        const float* z = z2 + (o / F) * F;
        const int k = o % F;
        float b = 0.f;
        for (int j = 0; j < F; ++j) b += z[j] * wh2[j * F + k];
        const float h = h1[i];
        dz1[i] = b * (1.f - h * h);
    }
}

// acc + the sum over p = p0 .. ascending of x[p * sx] * y[p * sy] (y null: of x alone), N preferences' loads in flight
// together; p0 moves behind the last whole batch
template <int N>
__device__ inline float trunk_dot_batches(float acc, int& p0, const float* __restrict__ x, int sx,
                                          const float* __restrict__ y, int sy, int P) {
    for (; p0 + N <= P; p0 += N) {
        float u[N], v[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            u[q] = x[(p0 + q) * sx];
            v[q] = y ? y[(p0 + q) * sy] : 1.f;
        }
#pragma unroll
        for (int q = 0; q < N; ++q) acc += u[q] * v[q];
    }
    return acc;
}
__device__ inline float trunk_dot(const float* x, int sx, const float* y, int sy, int P) {
    int p = 0;
    float a = trunk_dot_batches<32>(0.f, p, x, sx, y, sy, P);
    a = trunk_dot_batches<8>(a, p, x, sx, y, sy, P);
    return trunk_dot_batches<1>(a, p, x, sx, y, sy, P);
}

// Stage 2: dWh2, dbh2, dWh1, dbh1, one thread per output element.
__global__ __launch_bounds__(64) void k_hyper_trunk_bwd_b(const float* __restrict__ w, const float* __restrict__ h1,
                                                         const float* __restrict__ dz2, const float* __restrict__ dz1,
                                                         float* __restrict__ dhp, int P, int K, int F, int64_t o_wh1,
                                                         int64_t o_bh1, int64_t o_wh2, int64_t o_bh2) {
    int idx = blockIdx.x * 64 + threadIdx.x;
    if (idx < F * F) {
        dhp[o_wh2 + idx] = trunk_dot(dz2 + idx / F, F, h1 + idx % F, F, P);
        return;
    }
    idx -= F * F;
    if (idx < F * K) {
        dhp[o_wh1 + idx] = trunk_dot(dz1 + idx / K, F, w + idx % K, K, P);
        return;
    }
    idx -= F * K;
    if (idx < F) {
        dhp[o_bh2 + idx] = trunk_dot(dz2 + idx, F, nullptr, 0, P);
        return;
    }
    idx -= F;
    if (idx < F) dhp[o_bh1 + idx] = trunk_dot(dz1 + idx, F, nullptr, 0, P);
}

// Both stages in one workgroup, where its one CU reads the partials in less time than the second launch costs
// (trunk_bwd_inside).  The same sums.  LDS: dz2, dz1, h1 [P][F], w [P][K], the four shares [4][P F].
__global__ __launch_bounds__(1024) void k_hyper_trunk_bwd(const float* __restrict__ hp, const float* __restrict__ part, int n_chunk,
                                                         const float* __restrict__ f, const float* __restrict__ h1,
                                                         const float* __restrict__ w, float* __restrict__ dhp, int P, int K,
                                                         int F, int64_t o_wh1, int64_t o_bh1, int64_t o_wh2, int64_t o_bh2) {
    extern __shared__ float tl[];
    __shared__ float wh2[MORLAX_MAX_F * MORLAX_MAX_F];
    const int PF = P * F, tid = threadIdx.x;
    float *z2 = tl, *z1 = tl + PF, *sh = tl + 2 * PF, *red = tl + 3 * PF, *sw = tl + 7 * PF;
    for (int e = tid; e < F * F; e += 1024) wh2[e] = hp[o_wh2 + e];
    for (int e = tid; e < PF; e += 1024) sh[e] = h1[e];
    for (int e = tid; e < P * K; e += 1024) sw[e] = w[e];
    for (int e = tid; e < 4 * PF; e += 1024) {
        const float* src = part + e % PF;
        float a = 0.f;
        int c = e / PF;
        for (; c + 60 < n_chunk; c += 64) {  // sixteen chunks of this share per batch, loads in flight together
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = src[(int64_t)(c + 4 * u) * PF];
#pragma unroll
            for (int u = 0; u < 16; ++u) a += v[u];
        }
        for (; c + 12 < n_chunk; c += 16) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = src[(int64_t)(c + 4 * u) * PF];
#pragma unroll
            for (int u = 0; u < 4; ++u) a += v[u];
        }
        for (; c < n_chunk; c += 4) a += src[(int64_t)c * PF];
        red[e] = a;
    }
    __syncthreads();
    for (int i = tid; i < PF; i += 1024) {
        const float fv = f[i];
        z2[i] = (red[i] + red[PF + i] + red[2 * PF + i] + red[3 * PF + i]) * (1.f - fv * fv);
    }
    __syncthreads();
    for (int i = tid; i < PF; i += 1024) {
        const float* z = z2 + i / F * F;
        float b = 0.f;
        for (int j = 0; j < F; ++j) b += z[j] * wh2[j * F + i % F];
        z1[i] = b * (1.f - sh[i] * sh[i]);
    }
    __syncthreads();
    for (int e = tid; e < F * F + F * K + 2 * F; e += 1024) {
        int idx = e;
        const float *x, *y = nullptr;
        int sy = 0;
        float* dst;
        if (idx < F * F) {
            x = z2 + idx / F; y = sh + idx % F; sy = F; dst = dhp + o_wh2 + idx;
        } else if ((idx -= F * F) < F * K) {
            x = z1 + idx / K; y = sw + idx % K; sy = K; dst = dhp + o_wh1 + idx;
        } else if ((idx -= F * K) < F) {
            x = z2 + idx; dst = dhp + o_bh2 + idx;
        } else {
            idx -= F;
            x = z1 + idx; dst = dhp + o_bh1 + idx;
        }
        float a = 0.f;
        for (int p = 0; p < P; ++p) a += x[p * F] * (y ? y[p * sy] : 1.f);
        *dst = a;
    }
}

// Tiles, a wave each, of a dM workgroup: eight where there are enough, fewer so that few tiles still spread over the CUs
// (hypernet_bwd with 1 tile, with the rule, with 8: 100 preferences of 4 x 256, 210 tiles 75, 75 and 81 us; 128 of 4 x 512, 1073
// tiles 249, 235 and 236)
static int dm_tiles(int n_tiles) {
    const int t = (n_tiles + 127) / 128;
    return t < DMF_W ? t : DMF_W;
}

// Whether df workgroups request their chunk together.  Its 85 to 153 KB of LDS leave one workgroup a CU, the dM ones of the launch,
// which use none of it, included.  With up to 32 features the general form has room for two, so the whole chunk is for launches
// that are one round of one a CU; beyond, the registers hold the general form to one as well.  us a call of hypernet_bwd, tile by
// tile and chunk by chunk, 32 features: 24 preferences of 3 x 256 (159 workgroups) 35.8 and 32.5, 64 (206) 44.2 and 42.8, 64 of 2 x 160,
// strictly affine (238) 20.9 and 19.9, 48 of 3 x 384 (274) 56.8 and 59.0, 64 (317) 72.2 and 74.2, 32 of 3 x 512 (317) 62.0 and 63.0,
// 64 of 4 x 512 (402) 105.7 and 107.9; 64 features: 24 of 3 x 256 41.9 and 37.2, 8 of 4 x 512 66.2 and 60.5, 64 121.0 and 119.9.
static bool dm_df_brief(int F, int tiles_per_chunk, int workgroups) {
    return tiles_per_chunk == DMF_TB && (F > 32 || workgroups <= cu_count());
}

void launch_hypernet_bwd(const morlax_ctx* c, int net, const float* hparams, const float* w,
                         const float* dtheta_mat, const float* dtheta_vec, float* dhparams, void* ws,
                         bool kept, hipStream_t s) {
    const NetDev& nd = c->net[net];
    const AffineTable& at = c->aff[net];
    const int P = c->d.P, F = c->d.hyper_width, r = c->d.rank, K = c->d.K;
    HyperWs L = hyper_ws_layout(c, ws, nullptr);
    const bool affine = r < 0;
    // the gradient of the leading stacked rows: of the factor vector, or (strictly affine form) of theta_mat itself
    const float* dlead = affine ? dtheta_mat : L.dfac;
    // kept: the workspace still holds what the forward pass of this network left there (h1, f, the factors)
    if (affine) {
        // only f is needed again; dW0 and dMW come out of the dM pass below (W0 is the constant term of those rows)
        if (!kept)
            k_hyper_trunk<<<P, 64, 0, s>>>(trunk_of(c, net, w, L), hparams, F);
    } else {
        // recompute f and the factors; the theta_vec rows of the affine map land in a scratch nobody reads
        if (!kept) run_trunk_and_affine(c, net, hparams, w, L, L.vecs, s);
    }
    const int n_hidden = nd.n_layers - 1;
    auto elems = [&](int l) { return nd.layer[l].d_out * nd.layer[l].d_in; };
    BaseWork bw = {dhparams, nd.mat_len, layer_items(elems(0), n_hidden > 1 ? elems(1) : 0), 0, 0, 0};
    const LayerRule lr = layer_rule(nd);
    const AffineRows ar = affine_rows(at, F);
    const int n_base = affine ? 0 : (int)((nd.mat_len / 4 + 255) / 256);  // (strictly affine form: W0 is a constant of the rows)
    if (r > 0) {
        int merged = 0, n_runs = 0;  // elements of the largest dA that is added up from column runs; column runs of all layers
        auto runs = [&](int l) { return (nd.layer[l].d_in + DAB_COLS - 1) / DAB_COLS; };
        for (int l = 0; l < nd.n_layers; ++l) {
            if (runs(l) > 1 && nd.layer[l].d_out * r > merged) merged = nd.layer[l].d_out * r;
            n_runs += runs(l);
        }
        bw.n = n_base;
        bw.n_dab = n_runs * P;
        int nb = bw.n_dab + n_base;
        if (bw.n_dab > (P <= 80 ? 9 : 7) * cu_count() / 2) {
            const int rows = (n_base + 7) / 8, all = rows + (bw.n_dab + 7) / 8;
            bw.share = n_base <= cu_count() ? (uint64_t)1 << 32 : ((uint64_t)rows << 32) / all;
            nb = 8 * all;
        }
        auto dab = [&](auto kernel) {
            kernel<<<nb, 256, 0, s>>>(lr, layer_items(runs(0), n_hidden > 1 ? runs(1) : 0), row_div(P), bw, dtheta_mat, L.fac, L.dfac,
                                      L.da_part, r, P, nd.fac_len);
        };
        if (r <= 16) dab(k_hyper_dAB<1>);
        else dab(k_hyper_dAB<2>);
        if (merged > 0)
            k_hyper_dA_merge<<<dim3((merged + 1023) / 1024, P, nd.n_layers), 256, 0, s>>>(nd, L.da_part, L.dfac, r, P);
    }
    if (r == 0) k_hyper_base<<<n_base, 256, 0, s>>>(lr, bw, dtheta_mat, P);
    const int n_tiles = (at.q_total + DMF_Q - 1) / DMF_Q, tpw = df_chunk_tiles(at.q_total);
    const int n_chunk = (n_tiles + tpw - 1) / tpw;
    const int n_p = (P + DMF_P - 1) / DMF_P, n_df = n_chunk * n_p, dm_t = dm_tiles(n_tiles), n_dm = (n_tiles + dm_t - 1) / dm_t;
    auto dM_df = [&](auto jt, auto fine, auto brief) {
        constexpr int JT = decltype(jt)::value;
        constexpr int SHORT = decltype(brief)::value;
        constexpr int TB = SHORT ? DMF_TB : 1, bytes = 4 * (TB * ((SHORT ? SHORT : DMF_P) * 68 + DMF_Q * (16 * JT + 16)) + (SHORT ? TB * DMF_Q : 16 * DMF_Q + 64));
        auto kernel = k_hyper_dM_df<JT, decltype(fine)::value, SHORT>;
        if (bytes > 64 * 1024) {
            static std::atomic<uint64_t> allowed{0};  // devices on which the kernel may take more LDS than the default (a bit each)
            int dev = 0;
            (void)hipGetDevice(&dev);
            const uint64_t bit = (uint64_t)1 << (dev & 63);
            if (!(allowed.load(std::memory_order_relaxed) & bit)) {
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
                allowed.fetch_or(bit, std::memory_order_relaxed);
            }
        }
        kernel<<<n_df + n_dm, 64 * DMF_W, bytes, s>>>(hparams, ar, L.f, dlead, dtheta_vec, dhparams, L.df_part, P, F, nd.fac_len,
                                                      nd.vec_len, n_tiles, tpw, n_p, n_df, dm_t);
    };
    auto pick = [&](auto fine, auto brief) {
        if (F <= 32) dM_df(std::integral_constant<int, 2>{}, fine, brief);
        else dM_df(std::integral_constant<int, 4>{}, fine, brief);
    };
    const bool brief = P <= 64 && dm_df_brief(F, tpw, n_df + n_dm);
    if (n_p > 1) pick(std::true_type{}, std::integral_constant<int, 0>{});
    else if (brief && P <= 32) pick(std::false_type{}, std::integral_constant<int, 32>{});
    else if (brief) pick(std::false_type{}, std::integral_constant<int, 64>{});
    else pick(std::false_type{}, std::integral_constant<int, 0>{});
    const int lds = (7 * P * F + P * K) * 4;  // (with the kernel's 16 KB at most 64)
    if (trunk_bwd_inside(P, F, n_chunk) && lds <= 48 * 1024) {
        k_hyper_trunk_bwd<<<1, 1024, lds, s>>>(hparams, L.df_part, n_chunk, L.f, L.h1, w, dhparams, P, K, F, nd.hp_wh1, nd.hp_bh1,
                                               nd.hp_wh2, nd.hp_bh2);
        return;
    }
    const int ppb = 64 / F;  // preferences per block (F <= 64)
    k_hyper_trunk_bwd_a<<<(P + ppb - 1) / ppb, 256, 0, s>>>(hparams, L.df_part, n_chunk, L.f, L.h1, L.dz2, L.dz1, P, F,
                                                           nd.hp_wh2);
    k_hyper_trunk_bwd_b<<<(F * F + F * K + 2 * F + 63) / 64, 64, 0, s>>>(w, L.h1, L.dz2, L.dz1, dhparams, P, K, F,
                                                                        nd.hp_wh1, nd.hp_bh1, nd.hp_wh2, nd.hp_bh2);
}
