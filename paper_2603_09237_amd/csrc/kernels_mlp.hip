// Grouped target-network forward and backward (paper Sec. III-C rollout and update phases,
// Sec. III-E for the tanh head): every preference p applies its own weights W_l(p) to its own rows.
//
// Rows of preference p in a selection {t0, t_cnt, j0, j_cnt} are numbered m = (t - t0) * j_cnt +
// (j - j0); their home in the time-major tensors is row (t * N + p * n_g + j).  Hidden activations
// live in compact [P][M][W] buffers of the GEMM input type T (fp32 or bf16).
//
// Hidden layers run on MFMA: a 256-thread workgroup owns a 128 x 128 output tile of one preference,
// both operands are staged through LDS as rows of four 16-byte chunks along the contraction axis
// (32 bf16 or 16 fp32 values per step) and each of the four waves accumulates a 64 x 64 sub-tile with
// v_mfma_f32_32x32x16_bf16, fp32 operands as sums of three bf16 values (split3).  Operands whose contraction axis is the slow
// axis in memory (W in the dX product, both operands of the dW product) are transposed on the way
// into LDS.  The skinny output layer (<= 16 columns) uses 16x16 MFMA tiles, straight from global
// memory in the forward pass and on rows staged through LDS for its dW; its dZ is plain vector code.
#include "fused_fwd.h"

void launch_mlp_fwd_bf16_act(const FwdArgs& a, int rt, int n_tiles, hipStream_t s);
void launch_mlp_fwd_bf16_save(const FwdArgs& a, int rt, int n_tiles, hipStream_t s);
void launch_mlp_fwd_f32_act(const FwdArgs& a, int rt, int n_tiles, hipStream_t s);
void launch_mlp_fwd_f32_save(const FwdArgs& a, int rt, int n_tiles, hipStream_t s);

#define BM 128
#define BN 128
#define GEMM_NCH 4         // 16-byte chunks of the contraction axis staged per step and operand row

enum { SRC_KCONTIG = 0, SRC_KSTRIDED = 1, SRC_X_KCONTIG = 2 };

// One GEMM operand: a [rows x kdim] matrix of which a workgroup stages 128 rows x NCH 16-byte chunks of
// the contraction axis per step.  FAST = every access is a full, aligned vector (the launcher checks
// the shapes): loads are branch-free, out-of-range rows are clamped to a valid row (their results are
// never stored) and out-of-range contraction indices are masked to zero.  !FAST = element-wise loads
// with bounds checks, used only where a dimension is odd (first layer with an odd observation width).
//
// LDS row of a staged tile: bf16, the chunks as they are; fp32, the three bf16 parts of the step's values one after the other
// (NCH * 8 bytes each).  112 bytes for the sixteen fp32 values of a step: the sixteen rows a fragment read serves at a time
// start in sixteen different groups of four banks.
template <typename T> constexpr int gemm_pitch(int nch) { return (sizeof(T) == 4 ? 3 * nch * 8 : nch * 16) + 16; }
template <typename T, int NCH>
__device__ inline void put_chunk(unsigned char* tile, int row, int chunk, const uint4& u) {
    if constexpr (sizeof(T) == 4) {
        uint2 part[3];
        split3(u, part);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(tile + row * gemm_pitch<T>(NCH) + q * NCH * 8 + chunk * 8) = part[q];
    } else {
        *reinterpret_cast<uint4*>(tile + row * gemm_pitch<T>(NCH) + chunk * 16) = u;
    }
}
template <typename T, int KIND, bool FAST, int NCH>
struct Operand {
    const void* base;  // T* (compact kinds) or float* (x kinds), already offset to preference p
    int64_t ld;        // compact: elements between consecutive slow-axis indices; x: obs_dim
    int rows, kdim;    // valid extent
    RowMap rm;
    int p;

    static constexpr int VE = Elems<T>::VE;
    static constexpr int PITCH = gemm_pitch<T>(NCH);
    static constexpr int CPT = NCH / 2;  // chunks per thread (128 * NCH / 256)
    static constexpr bool PAIR = (KIND == SRC_KSTRIDED && sizeof(T) == 2 && FAST);

    // FAST: byte offset of the thread's chunk i at contraction index 0, relative to `base`.  Per-preference
    // tensors stay far below 4 GiB (checked by the launcher), so 32-bit offsets on a wave-uniform base do.
    uint32_t voff[CPT];

    __device__ inline float elem(int r, int k) const {
        if (r >= rows || k >= kdim) return 0.f;
        if (KIND == SRC_KCONTIG) return to_f(reinterpret_cast<const T*>(base)[(int64_t)r * ld + k]);
        if (KIND == SRC_KSTRIDED) return to_f(reinterpret_cast<const T*>(base)[(int64_t)k * ld + r]);
        return reinterpret_cast<const float*>(base)[rm.row(p, r) * ld + k];
    }

    // thread -> (tile row, chunk) of its i-th chunk
    __device__ static inline int trow(int i) {
        const int tid = threadIdx.x;
        if (KIND == SRC_KCONTIG || KIND == SRC_X_KCONTIG) return (tid + 256 * i) / NCH;
        if (PAIR) return 2 * (tid % 64);
        return tid % 128;
    }
    __device__ static inline int tchunk(int i) {
        const int tid = threadIdx.x;
        if (KIND == SRC_KCONTIG || KIND == SRC_X_KCONTIG) return (tid + 256 * i) % NCH;
        if (PAIR) return tid / 64 + 4 * (i / 2);  // chunks 2i and 2i+1 of a pair thread share the k range
        return tid / 128 + 2 * i;
    }

    __device__ inline void init(int r0) {
        if (!FAST) return;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            int r = r0 + trow(i);
            const int lim = PAIR ? rows - 2 : rows - 1;
            r = r < lim ? r : lim;
            if (KIND == SRC_KCONTIG) voff[i] = (uint32_t)(r * (int)ld + tchunk(i) * VE) * (uint32_t)sizeof(T);
            else if (KIND == SRC_X_KCONTIG) voff[i] = (uint32_t)((rm.row(p, r) * ld + tchunk(i) * VE) * 4);
            else voff[i] = (uint32_t)((tchunk(i) * VE * (int)ld + r) * (int)sizeof(T));
        }
    }

    // Raw staging registers per thread: the loads of step k+1 are issued before the products of step k
    // and nothing touches the loaded values until store(), so the load latency overlaps the MFMAs.
    static constexpr int RPC = (KIND == SRC_X_KCONTIG && sizeof(T) == 2) ? 2 : 1;  // uint4 registers per chunk (fp32 source of bf16)
    static constexpr int NRAW = FAST ? CPT * RPC : CPT;

    // Issue the loads of contraction range [k0, k0 + NCH * VE).  TAIL = the range may cross kdim: indices
    // are clamped (and the values masked in store()); otherwise addresses are base + uniform + voff.
    template <bool TAIL>
    __device__ inline void load(int r0, int k0, uint4 raw[NRAW]) const {
        if (!FAST) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int r = r0 + trow(i), k = k0 + tchunk(i) * VE;
                float v[8];
#pragma unroll
                for (int e = 0; e < VE; ++e) v[e] = elem(r, k + e);
                raw[i] = pack_chunk<T>(v);
            }
            return;
        }
        const char* b = reinterpret_cast<const char*>(base);
        if (KIND == SRC_KCONTIG || KIND == SRC_X_KCONTIG) {
            constexpr int ES = (KIND == SRC_KCONTIG) ? (int)sizeof(T) : 4;
            const char* bk = b + (int64_t)k0 * ES;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const char* src = bk + voff[i];
                if (TAIL && !(k0 + tchunk(i) * VE < kdim)) src = b + voff[i];  // any valid address; masked later
#pragma unroll
                for (int q = 0; q < RPC; ++q) raw[i * RPC + q] = reinterpret_cast<const uint4*>(src)[q];
            }
        } else {
            const int64_t rstep = ld * (int64_t)sizeof(T);  // bytes between consecutive k
            const char* bk = b + (int64_t)k0 * rstep;
#pragma unroll
            for (int i = 0; i < CPT; i += (PAIR ? 2 : 1)) {
                uint32_t d[8];
#pragma unroll
                for (int e = 0; e < (PAIR ? 8 : 4); ++e) {
                    const char* src = bk + e * rstep + voff[i];
                    if (TAIL) {
                        const int kk = k0 + tchunk(i) * VE + e;
                        if (kk >= kdim) src = b + (int64_t)(kdim - 1) * rstep + (voff[i] - (uint32_t)(tchunk(i) * VE) * (uint32_t)rstep);
                    }
                    d[e] = *reinterpret_cast<const uint32_t*>(src);
                }
                raw[i] = make_uint4(d[0], d[1], d[2], d[3]);
                if (PAIR) raw[i + 1] = make_uint4(d[4], d[5], d[6], d[7]);
            }
        }
    }

    // fp32, FAST: the same values through a buffer descriptor, zero beyond the contraction range (a 32-bit offset a request;
    // 64-bit addresses took the registers of a second step in flight)
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ inline void describe() {
        // K-strided tiles end with their last index; of the others an offset below the size of the tensor is asked for, or ~0
        const uint32_t n = KIND == SRC_KSTRIDED ? (uint32_t)kdim * (uint32_t)ld * 4u : 0xfffffff0u;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform_addr(base)), 0, (int)n, 0x00020000);
    }
    __device__ inline void request(int k0, uint4 raw[NRAW]) const {
        static_assert(!(FAST && sizeof(T) == 4) || NRAW == CPT, "one register quad a chunk");
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            if (KIND == SRC_KSTRIDED) {
                uint32_t d[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)  // (a preference's operand stays below 2 GiB: no offset wraps)
                    d[e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(voff[i] + (uint32_t)(k0 + e) * ((uint32_t)ld * 4u)), 0, 0);
                raw[i] = make_uint4(d[0], d[1], d[2], d[3]);
            } else {
                const uint32_t at = k0 + tchunk(i) * VE < kdim ? voff[i] + (uint32_t)k0 * 4u : 0xffffffffu;
                raw[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0));
            }
        }
    }

    __device__ static inline uint4 mask4(const uint4& u, bool ok) {
        const uint32_t m = ok ? 0xffffffffu : 0u;
        return make_uint4(u.x & m, u.y & m, u.z & m, u.w & m);
    }

    // Convert / transpose (and with TAIL mask) the staged values of range k0 and write them to the LDS tile.
    template <bool TAIL>
    __device__ inline void store(unsigned char* tile, const uint4 raw[NRAW], int k0) const {
        if (!FAST || KIND == SRC_KCONTIG) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const bool ok = !FAST || !TAIL || (k0 + tchunk(i) * VE < kdim);
                put_chunk<T, NCH>(tile, trow(i), tchunk(i), mask4(raw[i], ok));
            }
        } else if (PAIR) {
#pragma unroll
            for (int i = 0; i < CPT; i += 2) {
                const int k = k0 + tchunk(i) * 8;
                uint32_t d[8] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w, raw[i + 1].x, raw[i + 1].y, raw[i + 1].z, raw[i + 1].w};
                if (TAIL) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) d[e] = (k + e < kdim) ? d[e] : 0u;
                }
                const uint4 lo = make_uint4((d[0] & 0xffffu) | (d[1] << 16), (d[2] & 0xffffu) | (d[3] << 16),
                                            (d[4] & 0xffffu) | (d[5] << 16), (d[6] & 0xffffu) | (d[7] << 16));
                const uint4 hi = make_uint4((d[0] >> 16) | (d[1] & 0xffff0000u), (d[2] >> 16) | (d[3] & 0xffff0000u),
                                            (d[4] >> 16) | (d[5] & 0xffff0000u), (d[6] >> 16) | (d[7] & 0xffff0000u));
                *reinterpret_cast<uint4*>(tile + trow(i) * PITCH + tchunk(i) * 16) = lo;
                *reinterpret_cast<uint4*>(tile + (trow(i) + 1) * PITCH + tchunk(i) * 16) = hi;
            }
        } else if (KIND == SRC_KSTRIDED) {  // fp32, element-wise mask of the contraction tail
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int k = k0 + tchunk(i) * 4;
                uint4 u = raw[i];
                if (TAIL)
                    u = make_uint4(k < kdim ? u.x : 0u, k + 1 < kdim ? u.y : 0u, k + 2 < kdim ? u.z : 0u,
                                   k + 3 < kdim ? u.w : 0u);
                put_chunk<T, NCH>(tile, trow(i), tchunk(i), u);
            }
        } else {  // x source: fp32 -> T, whole chunks in or out of the contraction range
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const bool ok = !TAIL || (k0 + tchunk(i) * VE < kdim);
                float v[8];
#pragma unroll
                for (int q = 0; q < RPC; ++q) {
                    const uint4 u = raw[i * RPC + q];
                    v[4 * q] = __uint_as_float(u.x); v[4 * q + 1] = __uint_as_float(u.y);
                    v[4 * q + 2] = __uint_as_float(u.z); v[4 * q + 3] = __uint_as_float(u.w);
                }
                put_chunk<T, NCH>(tile, trow(i), tchunk(i), mask4(pack_chunk<T>(v), ok));
            }
        }
    }
};

// ---- epilogues.  A lane owns, for each of its 8 "octets", row r and the eight consecutive columns
// c .. c+7 (c a multiple of 8).  compute() turns the accumulators into results (left in v[], used for
// the column sums) and packs what will be stored; flush() issues the stores.  The kernel calls
// compute() for all octets first and then all flush()es back to back, so that the pieces of a cache
// line leave the wave together. ---------------------------------------------------------------------
template <typename T, int ACT, bool SAVE>
struct EpiFwd {  // h = act(z + b) and, when SAVE, act'(z); compact [M][ld] stores
    const float* bias;  // [ld] of preference p
    T* H;               // compact, offset to p
    typename GradT<T>::type* G;  // used when SAVE
    int ld;
    static constexpr bool kColSum = false;
    static constexpr bool kAhead = false;
    float* part;  // unused
    struct Out { Pack8 h, g; };
    __device__ inline void compute(int r, int c, int n, float v[8], Out& o) const {
        (void)r; (void)n;  // ld is a multiple of 16, so an octet is never cut
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += bias[c + i];
        compute_biased(v, o);
    }
    __device__ inline void compute_biased(float v[8], Out& o) const {  // v already holds z + b
        float g[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) act_pair<T, ACT, false>(v[i], v[i], g[i]);
        o.h = pack8(v, (const T*)nullptr);
        if (SAVE) o.g = pack8(g, (const typename GradT<T>::type*)nullptr);
    }
    static constexpr bool kBias = true;  // the persistent kernel stages the tile's bias slice in LDS
    static constexpr bool kPrefetch = false;
    __device__ inline void flush(int r, int c, int n, const Out& o) const {
        (void)n;
        put8(H + (int64_t)r * ld + c, o.h);
        if (SAVE) put8(G + (int64_t)r * ld + c, o.g);
    }
    // row-contiguous stores through an LDS patch (see the kernel): arrays, element size, row-0 address
    static constexpr bool kStage = true;
    static constexpr bool kStagePers = true;
    static constexpr int kArrays = SAVE ? 2 : 1;
    static constexpr int kES = (int)sizeof(T);
    __device__ inline char* arr(int a) const { return a == 0 ? reinterpret_cast<char*>(H) : reinterpret_cast<char*>(G); }
    __device__ static inline const Pack8& pk(const Out& o, int a) { return a == 0 ? o.h : o.g; }
};
template <typename T>
struct EpiDx {  // dZ_{l-1} = (dZ_l W_l) * act'(z_{l-1})
    const typename GradT<T>::type* G;
    T* dZ;
    int ld;
    static constexpr bool kColSum = true;  // column sums of the unrounded dZ feed the bias gradient
    float* part;                           // [P][tiles_m][ld] partial column sums
    struct Out { Pack8 d; };
    // the derivatives of an octet, requested together with those of the lane's other octets: one round trip a tile
    static constexpr bool kAhead = true;
    __device__ inline void request(int r, int c, Pack8& g) const {
        const uint4* src = reinterpret_cast<const uint4*>(G + (int64_t)r * ld + c);
        g.lo = src[0];
    }
    __device__ inline void compute_ahead(const Pack8& q, float v[8], Out& o) const {  // (bf16; fp32: epilogue_f32)
        float g[8];
        unpack8(q.lo, g);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= g[i];
        o.d = pack8(v, (const T*)nullptr);
    }
    __device__ inline void flush(int r, int c, int n, const Out& o) const {
        (void)n;
        put8(dZ + (int64_t)r * ld + c, o.d);
    }
    // the persistent kernel (bf16) fetches the derivatives of a 32-row block one block ahead of their use
    static constexpr bool kPrefetch = std::is_same<T, bf16_t>::value;
    __device__ inline uint4 fetch(int r, int c) const { return *reinterpret_cast<const uint4*>(G + (int64_t)r * ld + c); }
    __device__ inline void compute_fetched(const uint4& gq, float v[8], Out& o) const {
        float g[8];
        unpack8(gq, g);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= g[i];
        o.d = pack8(v, (const T*)nullptr);
    }
    static constexpr bool kStage = false;  // direct 16-byte stores measured faster in the 128 x 128 kernels,
    static constexpr bool kStagePers = true;  // row-contiguous staged stores in the persistent one
    static constexpr bool kBias = false;
    static constexpr int kArrays = 1;
    static constexpr int kES = (int)sizeof(T);
    __device__ inline char* arr(int) const { return reinterpret_cast<char*>(dZ); }
    __device__ static inline const Pack8& pk(const Out& o, int) { return o.d; }
};
struct EpiDw {  // dW_l(p)[o, i]
    float* dW;
    int ld;
    static constexpr bool kColSum = false;
    static constexpr bool kAhead = false;
    float* part;  // unused
    struct Out { Pack8 w; };
    __device__ inline void compute(int r, int c, int n, float v[8], Out& o) const {
        (void)r; (void)c; (void)n;
        o.w = pack8(v, (const float*)nullptr);
    }
    __device__ inline void flush(int r, int c, int n, const Out& o) const {
        float* d = dW + (int64_t)r * ld + c;
        if (n == 8 && (ld & 3) == 0) {
            put8(d, o.w);
        } else {
            const uint32_t w[8] = {o.w.lo.x, o.w.lo.y, o.w.lo.z, o.w.lo.w, o.w.hi.x, o.w.hi.y, o.w.hi.z, o.w.hi.w};
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < n) d[i] = __uint_as_float(w[i]);
        }
    }
    static constexpr bool kStage = false;
    static constexpr bool kStagePers = false;
    static constexpr bool kBias = false;
    static constexpr bool kPrefetch = false;
    static constexpr int kArrays = 1;
    static constexpr int kES = 4;
    __device__ inline char* arr(int) const { return reinterpret_cast<char*>(dW); }
    __device__ static inline const Pack8& pk(const Out& o, int) { return o.w; }
};

template <typename T, int ACT, bool SAVE>
__device__ inline void shift_epi(EpiFwd<T, ACT, SAVE>& e, int p, int64_t s0, int64_t s1, int64_t) {
    e.bias += (int64_t)p * s0;
    e.H += (int64_t)p * s1;
    if (SAVE) e.G += (int64_t)p * s1;
}
template <typename T> __device__ inline void shift_epi(EpiDx<T>& e, int p, int64_t s0, int64_t, int64_t) {
    e.G += (int64_t)p * s0;
    e.dZ += (int64_t)p * s0;
}
__device__ inline void shift_epi(EpiDw& e, int p, int64_t s0, int64_t, int64_t) { e.dW += (int64_t)p * s0; }

// One step of the pairwise fold of per-lane slot arrays: lanes whose bit H of lr is set keep the upper H
// slots, the others the lower H, and each adds what its partner (lr ^ H) held for the kept slots.
template <int H>
__device__ inline void fold_slots(float* cs, int lr) {
    const bool up = (lr & H) != 0;
#pragma unroll
    for (int t = 0; t < H; ++t) {
        const float send = up ? cs[t] : cs[t + H];
        const float keep = up ? cs[t + H] : cs[t];
        cs[t] = keep + __shfl_xor(send, H, 64);
    }
}

// ---- epilogue shared by the grouped GEMM kernels.  `lds0` is the workgroup's LDS, free for reuse (at
// least 36 KB); all four waves call this after a barrier.
template <class Epi>
__device__ inline void gemm_epilogue(const Epi& epi, float16_t (&acc)[2][2], unsigned char* lds0, int p, int tm,
                                     int tiles_m, int r0, int c0, int rows, int cols) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int lr = lane & 31, lg = lane >> 5;
    // The products were issued with the operands swapped, so each 32x32 accumulator holds the transposed
    // tile: lane (lr, lg) owns output row lr; with the row permutation of the B fragments its 16 values
    // are the columns 16 h + 8 lg + 0..7 for h = 0, 1 (accumulator elements 8 h .. 8 h + 7) -- one 16-byte
    // bf16 access per octet, and the two lane groups of a row together fill 32 contiguous bytes.
    float cs[Epi::kColSum ? 32 : 1];
    // kStage epilogues send their stores through a per-wave LDS patch (32 rows x 64 columns) so that every
    // store instruction writes whole 128-byte (bf16) or 256-byte (fp32) row segments instead of 32 bytes in
    // each of 32 rows; with two output arrays per tile that measured faster, with one it did not.
    constexpr int ES = Epi::kES;
    constexpr int WP = 64 * ES + 16;            // patch pitch in bytes
    constexpr int PPR = 64 * ES / 16;           // 16-byte pieces per patch row
    constexpr int NB = Epi::kStage ? 4 : 2;     // octets computed before their stores are issued
    unsigned char* patch = lds0 + wave * (32 * WP);
    Pack8 ahead[Epi::kAhead ? 2 : 1][Epi::kAhead ? 4 : 1];
    if constexpr (Epi::kAhead) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const int r = r0 + wm + 32 * i + lr, c = c0 + wn + 16 * o + 8 * lg;
                epi.request(r < rows ? r : rows - 1, c < cols ? c : 0, ahead[i][o]);
            }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = r0 + wm + 32 * i + lr;
#pragma unroll
        for (int jb = 0; jb < 4 / NB; ++jb) {
            typename Epi::Out outs[NB];
#pragma unroll
            for (int o = 0; o < NB; ++o) {
                const int j = (NB == 4) ? (o >> 1) : jb, h = o & 1;
                const int c = c0 + wn + 32 * j + 16 * h + 8 * lg;
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = acc[i][j][8 * h + u];
                const bool ok = (r < rows) && (c < cols);
                // out-of-range octets are computed on a clamped, valid position and not stored
                const int rc = r < rows ? r : rows - 1;
                const int cc = c < cols ? c : 0;
                if constexpr (Epi::kAhead) epi.compute_ahead(ahead[i][NB == 4 ? o : 2 * jb + o], v, outs[o]);
                else epi.compute(rc, cc, 8, v, outs[o]);
                if (Epi::kColSum) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int t = Epi::kColSum ? (16 * j + 8 * h + u) : 0;
                        cs[t] = (i == 0 ? 0.f : cs[t]) + (ok ? v[u] : 0.f);
                    }
                }
            }
            if (Epi::kStage) {
#pragma unroll
                for (int a = 0; a < Epi::kArrays; ++a) {
#pragma unroll
                    for (int o = 0; o < NB; ++o) {
                        unsigned char* dst = patch + lr * WP + (32 * (o >> 1) + 16 * (o & 1) + 8 * lg) * ES;
                        const Pack8& pk = Epi::pk(outs[o], a);
                        *reinterpret_cast<uint4*>(dst) = pk.lo;
                        if (ES == 4) *reinterpret_cast<uint4*>(dst + 16) = pk.hi;
                    }
                    __builtin_amdgcn_wave_barrier();
                    char* base = epi.arr(a);
#pragma unroll
                    for (int it = 0; it < 32 * PPR / 64; ++it) {
                        const int q = it * 64 + lane, prow = q / PPR, pc = q % PPR;
                        const uint4 u = *reinterpret_cast<const uint4*>(patch + prow * WP + pc * 16);
                        const int gr = r0 + wm + 32 * i + prow, gc = c0 + wn + pc * (16 / ES);
                        if (gr < rows && gc < cols)
                            *reinterpret_cast<uint4*>(base + ((int64_t)gr * epi.ld + gc) * ES) = u;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            } else {
#pragma unroll
                for (int o = 0; o < NB; ++o) {
                    const int c = c0 + wn + 32 * jb + 16 * (o & 1) + 8 * lg;
                    if (r < rows && c < cols) epi.flush(r, c, (cols - c < 8) ? (cols - c) : 8, outs[o]);
                }
            }
        }
    }
    if (Epi::kColSum) {
        // Column sums over the tile's 128 rows, fixed order.  Slot t = 16 j + 8 h + u of a lane is column
        // wn + 32 j + 16 h + 8 lg + u; the 32 lanes of a half-wave (same lg) fold their 32 slots pairwise so
        // that lane lr ends up with the half-wave total of slot lr.
        fold_slots<16>(cs, lr);
        fold_slots<8>(cs, lr);
        fold_slots<4>(cs, lr);
        fold_slots<2>(cs, lr);
        fold_slots<1>(cs, lr);
        float* red = reinterpret_cast<float*>(lds0 + 4 * 32 * WP);  // behind the store patches
        {
            const int j = lr >> 4, h = (lr >> 3) & 1, u = lr & 7;
            red[wave * 64 + 32 * j + 16 * h + 8 * lg + u] = cs[0];
        }
        __syncthreads();
        if (threadIdx.x < 128) {
            const int wsel = threadIdx.x >> 6, col = threadIdx.x & 63;
            const float v = red[wsel * 64 + col] + red[(2 + wsel) * 64 + col];
            if (c0 + threadIdx.x < cols)
                epi.part[((int64_t)p * tiles_m + tm) * epi.ld + c0 + threadIdx.x] = v;
        }
    }
}

// ---- epilogue of the fp32 products, and of fp32 results of bf16 ones.  Their operands are not swapped: lane (lr, lg) of a 32 x 32
// block holds column lr of the rows 8 (e / 4) + 4 lg + e % 4, so that an access of a wave is two whole 128-byte lines.  (As above, a row and eight columns a lane:
// 64 pieces of 16 bytes an access.  16 preferences x 8192 rows x 256 x 256, dX, which loads act' and stores dZ: 144 us, of which
// 60 were the epilogue's.  dW of bf16 operands, us a launch: 128 preferences x 2048 x 512 x 512 174.5 -> 166.5, 32 x 8192 x 256 x 256
// 65 -> 63, 24 x 1250 x 256 x 256 15.1 -> 14.4.)  Rows and columns beyond the edge fall to the buffer descriptors' bounds: their loads give zero,
// their stores do nothing.
struct TileF32 {
    uint32_t at;   // byte offset of the lane's element of row 0 of the block; beyond every tensor where its column is
    uint32_t ld4;  // bytes per row
    __device__ inline TileF32(int r, int c, int cols, int ld)
        : at(c < cols ? (uint32_t)(r * ld + c) * 4u : 0x80000000u), ld4((uint32_t)ld * 4u) {}
    __device__ static inline int row(int e) { return 8 * (e >> 2) + (e & 3); }
    __device__ inline int off(int e) const { return (int)(at + (uint32_t)row(e) * ld4); }
    // (a preference's tensor stays below 2 GiB)
    __device__ static inline __amdgpu_buffer_rsrc_t tensor(const float* base, int rows, int ld) {
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform_addr(base)), 0, rows * ld * 4, 0x00020000);
    }
    __device__ inline void put(__amdgpu_buffer_rsrc_t t, int e, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), t, off(e), 0, 0);
    }
    __device__ inline float get(__amdgpu_buffer_rsrc_t t, int e) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(t, off(e), 0, 0));
    }
};
// NI x NJ blocks of a wave at (r, c); `red`: 128 floats of LDS, used by the whole workgroup of four waves where the epilogue
// has column sums
template <typename T, int ACT, bool SAVE, int NI, int NJ>
__device__ inline void epilogue_f32(const EpiFwd<T, ACT, SAVE>& epi, float16_t (&acc)[NI][NJ], float*, int, int, int, int r, int c,
                                    int rows, int cols) {
    const int lr = threadIdx.x & 31, lg = (threadIdx.x >> 5) & 1;
    const auto H = TileF32::tensor(reinterpret_cast<const float*>(epi.H), rows, epi.ld);
    const auto G = TileF32::tensor(reinterpret_cast<const float*>(SAVE ? (const void*)epi.G : (const void*)epi.H), rows, epi.ld);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = c + 32 * j + lr;
        const float b = epi.bias[col < cols ? col : 0];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const TileF32 t(r + 32 * i + 4 * lg, col, cols, epi.ld);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float h, g;
                act_pair<T, ACT, false>(acc[i][j][e] + b, h, g);
                t.put(H, e, h);
                if (SAVE) t.put(G, e, g);
            }
        }
    }
}
template <int NI, int NJ>
__device__ inline void epilogue_f32(const EpiDw& epi, float16_t (&acc)[NI][NJ], float*, int, int, int, int r, int c, int rows, int cols) {
    const int lr = threadIdx.x & 31, lg = (threadIdx.x >> 5) & 1;
    const auto D = TileF32::tensor(epi.dW, rows, epi.ld);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const TileF32 t(r + 32 * i + 4 * lg, c + 32 * j + lr, cols, epi.ld);
#pragma unroll
            for (int e = 0; e < 16; ++e) t.put(D, e, acc[i][j][e]);
        }
}
template <int NI, int NJ>
__device__ inline void epilogue_f32(const EpiDx<float>& epi, float16_t (&acc)[NI][NJ], float* red, int p, int tm, int tiles_m, int r, int c,
                                    int rows, int cols) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
    const auto G = TileF32::tensor(epi.G, rows, epi.ld), D = TileF32::tensor(epi.dZ, rows, epi.ld);
    float16_t g[NI][NJ];  // all on their way together
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const TileF32 t(r + 32 * i + 4 * lg, c + 32 * j + lr, cols, epi.ld);
#pragma unroll
            for (int e = 0; e < 16; ++e) g[i][j][e] = t.get(G, e);
        }
    float part[NJ][4];  // (short chains: a quarter of the lane's rows each)
#pragma unroll
    for (int j = 0; j < NJ; ++j) part[j][0] = part[j][1] = part[j][2] = part[j][3] = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int row0 = r + 32 * i + 4 * lg;
            const TileF32 t(row0, c + 32 * j + lr, cols, epi.ld);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = acc[i][j][e] * g[i][j][e];
                t.put(D, e, v);
                part[j][e & 3] += row0 + TileF32::row(e) < rows ? v : 0.f;
            }
        }
    float sum[NJ];
    // column sums over the tile's 128 rows: lane groups, then the two waves above each other
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        sum[j] = (part[j][0] + part[j][1]) + (part[j][2] + part[j][3]);
        sum[j] += __shfl_xor(sum[j], 32, 64);
        if (wave >= 2 && lg == 0) red[(wave & 1) * 64 + 32 * j + lr] = sum[j];
    }
    __syncthreads();
    if (wave < 2 && lg == 0) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int col = c + 32 * j + lr;
            if (col < cols) epi.part[((int64_t)p * tiles_m + tm) * epi.ld + col] = sum[j] + red[wave * 64 + 32 * j + lr];
        }
    }
}

template <typename T, int KA, int KB, class Epi, bool FAST, int NCH>
struct GemmArgs {
    Operand<T, KA, FAST, NCH> a;
    Operand<T, KB, FAST, NCH> b;
    Epi epi;
    int64_t a_pstride, b_pstride;  // per-preference strides (elements of the operand's storage type)
    int64_t e0_pstride, e1_pstride, e2_pstride;
    int tiles_m, tiles_n;
    int crows = 0, ccols = 0;  // extent of the product (0: rows of a, rows of b)
    // dW with few preferences: the contraction cut into `ranges` pieces of `range` indices (a multiple of 64, the last
    // one shorter), each a group of its own: group p * ranges + s multiplies range s of preference p
    int ranges = 1, range = 0;

    struct Group { int p, k0, kdim; };  // preference, first contraction index, contraction length
    __device__ inline Group group(int id) const {
        if (KA != SRC_KSTRIDED || KB != SRC_KSTRIDED || ranges == 1) return {id, 0, a.kdim};
        const int pp = id / ranges, k0 = (id - pp * ranges) * range;
        return {pp, k0, a.kdim - k0 < range ? a.kdim - k0 : range};
    }
    // base of the operands for a group (compact kinds; k0 > 0 only where the contraction axis is the slow one)
    __device__ inline const T* a_base(const Group& q) const {
        return reinterpret_cast<const T*>(a.base) + (int64_t)q.p * a_pstride + (int64_t)q.k0 * a.ld;
    }
    __device__ inline const T* b_base(const Group& q) const {
        return reinterpret_cast<const T*>(b.base) + (int64_t)q.p * b_pstride + (int64_t)q.k0 * b.ld;
    }
};

// One 32 x 32 block of an fp32 product once more, on the fp32 matrix instructions and from memory: what is left to do where
// the sums of split operands came out undefined or infinite (see split3: an infinite operand does that).  It is the exception, and
// short code: sixteen indices requested together take a backward pass of 16 preferences x 8192 rows of 3 x 256 with an undefined
// value from 1850 to 1510 us (660 without one), and every other pass 0.4 - 0.8 % longer.
template <class OpA, class OpB>
__device__ inline void plain_products(const OpA& A, const OpB& B, int r, int c, int kdim, float16_t& acc) {
    const int lg = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll 1
    for (int k = 0; k < kdim; k += 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A.elem(r, k + lg), B.elem(c, k + lg), acc, 0, 0, 0);
}

// C[rows_a x rows_b] = A[rows_a x K] * B[rows_b x K]^T for every preference.  fp32 on split operands, us a launch, 16 preferences x
// 8192 rows x 256 x 256: dX 203 -> 120 (of which the loop is 72; its products alone 43 at the matrix pipe's rate), dW 165 -> 96.
template <typename T, int KA, int KB, class Epi, bool FAST, int NCH>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 2 : 1) void k_grouped_gemm(GemmArgs<T, KA, KB, Epi, FAST, NCH> g) {
    constexpr int PITCH = gemm_pitch<T>(NCH);
    constexpr int TILE = 128 * PITCH;
    constexpr bool SPLIT = sizeof(T) == 4;
    __shared__ __align__(16) unsigned char lds[2][2][TILE];
    constexpr int VE = Elems<T>::VE;
    constexpr int BK = NCH * VE;
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int per_p = g.tiles_m * g.tiles_n;
    const int p = id / per_p, tm = (id % per_p) / g.tiles_n, tn = id % g.tiles_n;

    Operand<T, KA, FAST, NCH> A = g.a;
    Operand<T, KB, FAST, NCH> B = g.b;
    const auto grp = g.group(p);
    A.p = p; B.p = p;
    if (KA == SRC_KCONTIG || KA == SRC_KSTRIDED) A.base = g.a_base(grp);
    if (KB == SRC_KCONTIG || KB == SRC_KSTRIDED) B.base = g.b_base(grp);
    A.kdim = B.kdim = grp.kdim;
    Epi epi = g.epi;
    shift_epi(epi, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);

    const int r0 = tm * BM, c0 = tn * BN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int lr = lane & 31, lg = lane >> 5;
    // B rows are fed to the MFMA with bits 2 and 3 of the row index swapped, which makes every lane's
    // accumulators cover two runs of eight consecutive output columns (see the epilogue)
    const int lrp = (lr & 0x13) | ((lr & 4) << 1) | ((lr & 8) >> 1);
    A.init(r0);
    B.init(c0);

    float16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    float16_t low[SPLIT ? 2 : 1][2];  // fp32: the products of the smaller parts
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) low[i][j] = acc[i][j];
    }

    const int kdim = A.kdim;
    const int nk = (kdim + BK - 1) / BK;
    constexpr int NRA = Operand<T, KA, FAST, NCH>::NRAW, NRB = Operand<T, KB, FAST, NCH>::NRAW;
    const int nfull = kdim / BK;  // steps [0, nfull) are entirely inside the contraction range
    if constexpr (SPLIT) {
        // Two steps are on their way in registers.  The older one is split and written to the other LDS stage between the
        // products of the step in LDS: 24 of them, 32 cycles each, against some 100 vector instructions.
        static_assert(!SPLIT || NCH == 4, "a step is one product deep");
        uint4 ra[2][NRA], rb[2][NRB];
        if constexpr (FAST) { A.describe(); B.describe(); }
        auto request = [&](int kt, auto set_tag) __attribute__((always_inline)) {
            constexpr int U = decltype(set_tag)::value;
            if constexpr (FAST) {
                A.request(kt * BK, ra[U]);
                B.request(kt * BK, rb[U]);
            } else {
                A.template load<true>(r0, kt * BK, ra[U]);
                B.template load<true>(c0, kt * BK, rb[U]);
            }
        };
        auto step = [&](int kt, auto set_tag) __attribute__((always_inline)) {
            constexpr int U = decltype(set_tag)::value;
            const unsigned char* ta = lds[U ^ 1][0] + (wm + lr) * PITCH + lg * 16;
            const unsigned char* tb = lds[U ^ 1][1] + (wn + lr) * PITCH + lg * 16;
            uint4 fa[2][3], fb[2][3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; i < 2; ++i) fa[i][q] = *reinterpret_cast<const uint4*>(ta + 32 * i * PITCH + q * 32);
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[j][q] = *reinterpret_cast<const uint4*>(tb + 32 * j * PITCH + q * 32);
            }
            A.template store<false>(lds[U][0], ra[U], 0);
            B.template store<false>(lds[U][1], rb[U], 0);
            request(kt + 3, set_tag);
#pragma unroll
            for (int t = 0; t < 6; ++t)  // (one round over all blocks a term: no product waits for the one before)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) split_mma(t, fa[i], fb[j], acc[i][j], low[i][j]);
            if (FAST) {
#pragma unroll
                for (int u = 0; u < 24; ++u) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a product,
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);  // vector instructions,
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // a write to LDS
                }
            }
            __syncthreads();
        };
        constexpr std::integral_constant<int, 0> even{};
        constexpr std::integral_constant<int, 1> odd{};
        request(0, even);
        request(1, odd);
        A.template store<false>(lds[0][0], ra[0], 0);
        B.template store<false>(lds[0][1], rb[0], 0);
        request(2, even);
        __syncthreads();
        for (int kt = 0; kt < nk; kt += 2) {
            step(kt, odd);
            if (kt + 1 < nk) step(kt + 1, even);
        }
    } else {
        // Register stage + two LDS stages: the loads of step kt+1 are in flight while step kt is multiplied
        // out of LDS; they are converted and written to the other LDS stage after the products.  Only the last
        // step can cross the end of the contraction range; it alone runs the clamped / masked loader.
        uint4 ra[NRA], rb[NRB];
        if (nfull > 0) {
            A.template load<false>(r0, 0, ra);
            B.template load<false>(c0, 0, rb);
            A.template store<false>(lds[0][0], ra, 0);
            B.template store<false>(lds[0][1], rb, 0);
        } else {
            A.template load<true>(r0, 0, ra);
            B.template load<true>(c0, 0, rb);
            A.template store<true>(lds[0][0], ra, 0);
            B.template store<true>(lds[0][1], rb, 0);
        }
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            const int cur = kt & 1;
            const bool more = kt + 1 < nk, full = kt + 1 < nfull;
            if (full) {
                A.template load<false>(r0, (kt + 1) * BK, ra);
                B.template load<false>(c0, (kt + 1) * BK, rb);
            } else if (more) {
                A.template load<true>(r0, (kt + 1) * BK, ra);
                B.template load<true>(c0, (kt + 1) * BK, rb);
            }
            const unsigned char* ta = lds[cur][0] + (wm + lr) * PITCH + lg * 16;
            const unsigned char* tb = lds[cur][1] + (wn + lrp) * PITCH + lg * 16;
#pragma unroll
            for (int ks = 0; ks < NCH / 2; ++ks) {
                uint4 fa[2], fb[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) fa[i] = *reinterpret_cast<const uint4*>(ta + 32 * i * PITCH + ks * 32);
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[j] = *reinterpret_cast<const uint4*>(tb + 32 * j * PITCH + ks * 32);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) Mma32<T>::run(fb[j], fa[i], acc[i][j]);  // transposed tile
            }
            if (full) {
                A.template store<false>(lds[cur ^ 1][0], ra, (kt + 1) * BK);
                B.template store<false>(lds[cur ^ 1][1], rb, (kt + 1) * BK);
            } else if (more) {
                A.template store<true>(lds[cur ^ 1][0], ra, (kt + 1) * BK);
                B.template store<true>(lds[cur ^ 1][1], rb, (kt + 1) * BK);
            }
            __syncthreads();
        }
    }
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[i][j] += low[i][j];
                if (any_undefined(acc[i][j])) plain_products(A, B, r0 + wm + 32 * i + lr, c0 + wn + 32 * j + lr, kdim, acc[i][j]);
            }
        epilogue_f32(epi, acc, reinterpret_cast<float*>(&lds[0][0][0]), p, tm, g.tiles_m, r0 + wm, c0 + wn, g.crows, g.ccols);
    } else {
        gemm_epilogue(epi, acc, &lds[0][0][0], p, tm, g.tiles_m, r0, c0, g.crows, g.ccols);
    }
}

// ---- bf16 grouped GEMM with direct-to-LDS loads ------------------------------------------------
// Same tiles, wave layout and epilogues as k_grouped_gemm, for bf16 operands whose shapes need no
// masking (the launcher checks them).  Operand tiles go from global memory straight into LDS, 16 bytes
// per lane, DMA_NST - 1 contraction steps ahead of the products, so that the latency of a load from HBM
// is covered by several steps of MFMAs instead of one.  A DMA instruction fills 1 KB of LDS, lane l
// writing bytes 16 l .. 16 l + 15 of it; which global chunk a lane fetches is free, and that is where
// the bank swizzles below are applied.
//   SRC_KCONTIG  operand, stage = 128 rows x 4 chunks (8 contraction indices each): chunk (r, c) sits at
//                position 4 r + (c ^ swz(r)); fragments are read with one 16-byte LDS read.
//   SRC_KSTRIDED operand (global [k][row]), stage = 32 k x 16 chunks (8 rows each): chunk (k, ic) sits at
//                position 16 k + (ic ^ 4 (k & 3)); fragments are read with two transposing 8-byte reads,
//                each of which hands lane b of a 16-lane group the elements [k0 .. k0+3][row b] of the
//                4 x 16 block whose 64-bit words the lanes 4 e + c (k = k0 + e, rows 4 c .. 4 c + 3) address.
#define DMA_NST 4
#define DMA_STAGE_BYTES 16384  // A tile 8 KB, then B tile 8 KB

typedef short short4_t __attribute__((ext_vector_type(4)));

// The LDS has 64 banks of 4 bytes: it serves 16 lanes of a 16-byte read, or 32 lanes of an 8-byte read,
// per cycle, and the lanes of such a group must touch distinct slots modulo 256 bytes.  With 64-byte rows,
// rows r .. r+3 fill one 256-byte window, so the chunk index is XORed with bits 2, 3 of the row; the
// K-strided tiles XOR bits 2, 3 of the chunk index with the contraction index modulo 4.
__device__ inline int swz_rk(int r) { return (r >> 2) & 3; }

template <int KIND>
struct DmaOperand {
    const char* base;   // per-preference base, bytes
    uint32_t voff[2];   // lane offsets of its two DMA instructions per stage
    int64_t kstep;      // bytes per contraction step (32 indices)
    uint32_t roff;      // lane's LDS byte offset of fragment (block 0, ks 0) within the operand's stage tile

    __device__ inline void init(const bf16_t* b, int ld, int rows, int t0, int wbase, bool brole) {
        base = reinterpret_cast<const char*>(b);
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int j = 2 * wave + i;
            if (KIND == SRC_KCONTIG) {
                const int row = 16 * j + lane / 4, c = (lane % 4) ^ swz_rk(row);
                int gr = t0 + row;
                gr = gr < rows ? gr : rows - 1;
                voff[i] = (uint32_t)((gr * ld + 8 * c) * 2);
            } else {
                const int k = 4 * j + lane / 16, ic = (lane % 16) ^ (4 * (k & 3));
                int gr = t0 + 8 * ic;
                gr = gr < rows - 8 ? gr : rows - 8;
                voff[i] = (uint32_t)((k * ld + gr) * 2);
            }
        }
        kstep = (KIND == SRC_KCONTIG) ? 64 : (int64_t)64 * ld;
        const int lr = lane & 31, lg = lane >> 5;
        if (KIND == SRC_KCONTIG) {
            const int rr = brole ? ((lr & 0x13) | ((lr & 4) << 1) | ((lr & 8) >> 1)) : lr;
            const int row = wbase + rr;
            roff = (uint32_t)(row * 64 + ((lg ^ swz_rk(row)) * 16));
        } else {
            const int a = lane & 15, q0 = (lane >> 4) & 1, e = a >> 2, c = a & 3;
            const int cs = brole ? (((c & 1) << 1) | (c >> 1)) : c;
            const int col = wbase + 16 * q0 + 4 * cs, k = 8 * lg + e;
            roff = (uint32_t)((k * 16 + ((col >> 3) ^ (4 * (k & 3)))) * 16 + ((col >> 2) & 1) * 8);
        }
    }
    // issue the loads of contraction step kt into the stage tile at LDS address `tile`
    __device__ inline void issue(int kt, uint32_t tile) const {
        const char* b = base + (int64_t)kt * kstep;
        const int wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            dma16(b, voff[i], __builtin_amdgcn_readfirstlane(tile + (uint32_t)(2 * wave + i) * 1024u));
    }
    // fragment of 32-row block `blk` (0, 1) for the 16 contraction indices ks (0, 1) of the stage
    __device__ inline uint4 frag(const unsigned char* tile, int blk, int ks) const {
        if (KIND == SRC_KCONTIG) {
            // chunk 2 ks + lg: the swizzle only touches the low two bits, so ks selects the upper half
            return *reinterpret_cast<const uint4*>(tile + ((roff + blk * 2048) ^ (uint32_t)(ks * 32)));
        } else {
            typedef __attribute__((address_space(3))) short4_t lds_s4;
            const uint32_t o = (roff ^ (uint32_t)(blk * 64)) + ks * 4096;
            const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(tile + o));
            const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(tile + o + 1024));
            uint2 a = __builtin_bit_cast(uint2, lo), b2 = __builtin_bit_cast(uint2, hi);
            return make_uint4(a.x, a.y, b2.x, b2.y);
        }
    }
};

// Epilogue of dX (bf16) on tiles of 64 MB x 64 STRIPS.  The derivatives of a 32-row block (32 x 64 codes, 4 KB a wave) come by
// direct-to-LDS loads of whole 128-byte row segments, two blocks ahead: fetched into registers as a lane needs them, 16 bytes of each of 64 rows a
// request, the vector cache looks up four times as many addresses.  Two patches a wave, `even` and `odd`, take a block's
// derivatives and then its results, which leave as whole row segments as well.  Requested so far: block 0 into `even`, behind
// it `behind` loads of the next tile's first stages.  us a launch, as it was and so: 128 preferences x 2048 x 512 x 512 232 and
// 219, 64 x 4096 x 512 x 512 257 and 232, 32 x 8192 x 256 x 256 93 and 82; on 128 x 128 tiles 24 x 1250 x 256 x 256 15.8 and 13.6.
struct DxBlocks {
    const char* G;  // of the preference
    int rows, ld2, row0;
    uint32_t col;
    // (r, c): the wave's first row and column.  Rows and columns beyond the edge repeat the last row, column 0 (their results are
    // not stored)
    __device__ inline DxBlocks(const EpiDx<bf16_t>& epi, int r, int c, int rows_, int cols) {
        const int lane = threadIdx.x & 63;
        G = reinterpret_cast<const char*>(epi.G);
        rows = rows_; ld2 = epi.ld * 2;
        row0 = r + (lane >> 3);
        const int cc = c + 8 * ((lane & 7) ^ (lane >> 3));  // piece c of row q of a block lies at c ^ (q & 7)
        col = (uint32_t)(cc < cols ? cc : 0) * 2u;
    }
    __device__ inline void request(int i, const unsigned char* patch) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = row0 + 32 * i + 8 * j;
            dma16(G, (uint32_t)((r < rows ? r : rows - 1) * ld2) + col,
                  __builtin_amdgcn_readfirstlane((uint32_t)(size_t)patch + (uint32_t)j * 1024u));
        }
    }
};
template <int MB, int STRIPS>
__device__ inline void dx_epilogue(const EpiDx<bf16_t>& epi, const DxBlocks& blocks, float16_t (&acc)[MB][2], unsigned char* even,
                                   unsigned char* odd, float* red, int behind, int p, int tm, int tiles_m, int r0, int c0, int rows, int cols,
                                   int wm, int wn) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
    // a tile inside the matrix stores four times a block, so that the loads behind the ones waited for can be counted
    const bool inside = r0 + 64 * MB <= rows && c0 + 64 * STRIPS <= cols;
    blocks.request(1, odd);
    float cs[32];
    char* base = reinterpret_cast<char*>(epi.dZ);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        unsigned char* patch = (i & 1) ? odd : even;
        if (!inside) wait_vm<0>();
        else if (i == 0) {  // behind block 0: the next tile's first stages, block 1
            if (behind == 8) wait_vm<12>();
            else if (behind == 0) wait_vm<4>();
            else wait_vm<0>();
        } else if (i + 1 < MB) wait_vm<8>();  // the stores of the block before, the loads of the block after
        else wait_vm<4>();
        const int r = r0 + wm + 32 * i + lr;
        uint4 gq[4];
#pragma unroll
        for (int o = 0; o < 4; ++o)
            gq[o] = *reinterpret_cast<const uint4*>(patch + lr * 128 + (((2 * o + lg) ^ (lr & 7)) * 16));
        typename EpiDx<bf16_t>::Out out[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const bool ok = inside || ((r < rows) && (c0 + wn + 16 * o + 8 * lg < cols));
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = acc[i][o >> 1][8 * (o & 1) + u];
            epi.compute_fetched(gq[o], v, out[o]);
#pragma unroll
            for (int u = 0; u < 8; ++u) cs[8 * o + u] = (i == 0 ? 0.f : cs[8 * o + u]) + (ok ? v[u] : 0.f);
        }
#pragma unroll
        for (int o = 0; o < 4; ++o) *reinterpret_cast<uint4*>(patch + lr * 128 + (((2 * o + lg) ^ (lr & 7)) * 16)) = out[o].d.lo;
        __builtin_amdgcn_wave_barrier();
        uint4 q[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int prow = it * 8 + (lane >> 3), pc = lane & 7;
            q[it] = *reinterpret_cast<const uint4*>(patch + prow * 128 + ((pc ^ (prow & 7)) * 16));
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int gr = r0 + wm + 32 * i + it * 8 + (lane >> 3), gc = c0 + wn + (lane & 7) * 8;
            if (inside || (gr < rows && gc < cols)) *reinterpret_cast<uint4*>(base + ((int64_t)gr * epi.ld + gc) * 2) = q[it];
        }
        __builtin_amdgcn_wave_barrier();
        // (the stores hold what was read from the patch, so it is free)
        if (i + 2 < MB) blocks.request(i + 2, patch);
    }
    // column sums, as in tile_epilogue
    fold_slots<16>(cs, lr);
    fold_slots<8>(cs, lr);
    fold_slots<4>(cs, lr);
    fold_slots<2>(cs, lr);
    fold_slots<1>(cs, lr);
    {
        const int j = lr >> 4, h = (lr >> 3) & 1, u = lr & 7;
        red[wave * 64 + 32 * j + 16 * h + 8 * lg + u] = cs[0];
    }
    __syncthreads();
    if (threadIdx.x < 64 * STRIPS) {  // the two waves of a 64-column strip: wave ids s and s + STRIPS
        const int strip = threadIdx.x >> 6, col = threadIdx.x & 63;
        const float v = red[strip * 64 + col] + red[(STRIPS + strip) * 64 + col];
        if (c0 + threadIdx.x < cols) epi.part[((int64_t)p * tiles_m + tm) * epi.ld + c0 + threadIdx.x] = v;
    }
}

template <int KA, int KB, class Epi>
__global__ __launch_bounds__(256) void k_gemm_dma(GemmArgs<bf16_t, KA, KB, Epi, true, GEMM_NCH> g) {
    extern __shared__ __align__(16) unsigned char dlds[];
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int per_p = g.tiles_m * g.tiles_n;
    const int p = id / per_p, tm = (id % per_p) / g.tiles_n, tn = id % g.tiles_n;
    Epi epi = g.epi;
    shift_epi(epi, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);
    const int r0 = tm * BM, c0 = tn * BN;
    const int wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    constexpr bool DX = std::is_same<Epi, EpiDx<bf16_t>>::value;
    constexpr bool LINES = std::is_same<Epi, EpiDw>::value;  // fp32 results: stored as whole lines (epilogue_f32)
    DmaOperand<KA> A;
    DmaOperand<KB> B;
    const auto grp = g.group(p);
    A.init(g.a_base(grp), (int)g.a.ld, g.a.rows, r0, wm, false);
    B.init(g.b_base(grp), (int)g.b.ld, g.b.rows, c0, wn, !LINES);

    float16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int nk = grp.kdim / 32;
    const uint32_t lbase = (uint32_t)(size_t)dlds;
#pragma unroll
    for (int st = 0; st < DMA_NST - 1; ++st)
        if (st < nk) {
            A.issue(st, lbase + st * DMA_STAGE_BYTES);
            B.issue(st, lbase + st * DMA_STAGE_BYTES + 8192);
        }
    for (int kt = 0; kt < nk; ++kt) {
        // each wave has 4 loads per stage in flight; the oldest stage is the one multiplied next
        const int ahead = nk - 1 - kt;
        if (ahead >= 2) wait_vm<8>();
        else if (ahead == 1) wait_vm<4>();
        else wait_vm<0>();
        __syncthreads();  // stage kt has landed for every wave, and everyone is done with stage kt - 1
        if (kt + DMA_NST - 1 < nk) {
            const uint32_t tile = lbase + (uint32_t)((kt + DMA_NST - 1) % DMA_NST) * DMA_STAGE_BYTES;
            A.issue(kt + DMA_NST - 1, tile);
            B.issue(kt + DMA_NST - 1, tile + 8192);
        }
        if constexpr (DX) {  // the epilogue's first block, into a stage that nobody reads any more
            if (kt == nk - 1)
                DxBlocks(epi, r0 + wm, c0 + wn, g.crows, g.ccols).request(0, dlds + (nk % DMA_NST) * DMA_STAGE_BYTES + wave * 4096);
        }
        const unsigned char* ta = dlds + (kt % DMA_NST) * DMA_STAGE_BYTES;
        const unsigned char* tb = ta + 8192;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            uint4 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[i] = A.frag(ta, i, ks);
#pragma unroll
            for (int j = 0; j < 2; ++j) fb[j] = B.frag(tb, j, ks);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (LINES) Mma32<bf16_t>::run(fa[i], fb[j], acc[i][j]);
                    else Mma32<bf16_t>::run(fb[j], fa[i], acc[i][j]);  // transposed tile
                }
        }
    }
    if constexpr (LINES) {
        epilogue_f32(epi, acc, nullptr, p, tm, g.tiles_m, r0 + wm, c0 + wn, g.crows, g.ccols);
    } else if constexpr (DX) {
        // (the stages of steps nk - 4, nk - 3 and nk - 2, which every wave has left)
        dx_epilogue<2, 2>(epi, DxBlocks(epi, r0 + wm, c0 + wn, g.crows, g.ccols), acc, dlds + (nk % DMA_NST) * DMA_STAGE_BYTES + wave * 4096,
                          dlds + ((nk + 1) % DMA_NST) * DMA_STAGE_BYTES + wave * 4096,
                          reinterpret_cast<float*>(dlds + ((nk + 2) % DMA_NST) * DMA_STAGE_BYTES), 0, p, tm, g.tiles_m, r0, c0, g.crows,
                          g.ccols, wm, wn);
    } else {
        __syncthreads();
        gemm_epilogue(epi, acc, dlds, p, tm, g.tiles_m, r0, c0, g.crows, g.ccols);
    }
}

// ---- persistent bf16 grouped GEMM, 256 x TN tiles -----------------------------------------------
// Resident workgroups walk over the tiles; a wave owns 128 x 64 outputs (4 x 2 blocks of 32 x 32, 128
// accumulator registers), which reads three quarters of the LDS bytes per product that the 64 x 64 wave
// tiles above read.  Operand stages (A 16 KB, B TN * 64 bytes) are filled by direct-to-LDS loads two
// contraction steps ahead, and the first two stages of a workgroup's next tile are requested before the
// epilogue of the current one, so that their latency is covered by the epilogue's arithmetic.  The
// layouts inside a stage follow DmaOperand; a row of a K-strided tile has ROWS / 8 chunks.
#define PG_NST 3
#define PG_A_BYTES 16384
#define PG_TM 256
// TN = 128: four waves (2 x 2), two workgroups per CU.  TN = 256: eight waves (2 x 4), one workgroup per CU;
// a third fewer operand bytes per product travel from the L2 into LDS.
template <int TN> struct PgShape {
    static constexpr int kWaves = TN / 32;                 // 128 x 64 outputs per wave
    static constexpr int kBBytes = TN * 64;
    static constexpr int kStage = PG_A_BYTES + kBBytes;
    static constexpr int kLds = PG_NST * kStage;
    static constexpr int kLoads = (PG_A_BYTES + kBBytes) / 1024 / kWaves;  // DMA instructions per wave and stage
};

template <int KIND, int ROWS, int MBLK, int NW>
struct DmaTile {
    static constexpr int NI = ROWS / 16 / NW;  // DMA instructions per wave and stage
    static constexpr int CPR = ROWS / 8;   // chunks per contraction index (K-strided layout)
    const char* base;
    uint32_t voff[NI];
    int64_t kstep;
    uint32_t roff[MBLK];  // LDS byte offset of the lane's fragment of block b, ks 0

    // K-strided tiles: what the chunk index is XORed with at contraction index k, so that the four consecutive indices of a
    // transposing read fall into different banks (eight chunks to an index: the neighbouring index already does)
    __device__ static inline int swz(int k) { return CPR >= 16 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); }
    __device__ inline void set_tile(const bf16_t* b, int ld, int rows, int t0) {
        base = reinterpret_cast<const char*>(b);
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int j = NI * wave + i;
            if (KIND == SRC_KCONTIG) {
                const int row = 16 * j + lane / 4, c = (lane % 4) ^ swz_rk(row);
                int gr = t0 + row;
                gr = gr < rows ? gr : rows - 1;
                voff[i] = (uint32_t)((gr * ld + 8 * c) * 2);
            } else {
                const int pos = 64 * j + lane, k = pos / CPR, ic = (pos % CPR) ^ swz(k);
                int gr = t0 + 8 * ic;
                gr = gr < rows - 8 ? gr : rows - 8;
                voff[i] = (uint32_t)((k * ld + gr) * 2);
            }
        }
        kstep = (KIND == SRC_KCONTIG) ? 64 : (int64_t)64 * ld;
    }
    __device__ inline void set_lane(int wbase, bool brole) {
        const int lane = threadIdx.x & 63, lr = lane & 31, lg = lane >> 5;
#pragma unroll
        for (int b = 0; b < MBLK; ++b) {
            if (KIND == SRC_KCONTIG) {
                const int rr = brole ? ((lr & 0x13) | ((lr & 4) << 1) | ((lr & 8) >> 1)) : lr;
                const int row = wbase + 32 * b + rr;
                roff[b] = (uint32_t)(row * 64 + ((lg ^ swz_rk(row)) * 16));
            } else {
                const int a = lane & 15, q0 = (lane >> 4) & 1, e = a >> 2, c = a & 3;
                const int cs = brole ? (((c & 1) << 1) | (c >> 1)) : c;
                const int col = wbase + 32 * b + 16 * q0 + 4 * cs, k = 8 * lg + e;
                roff[b] = (uint32_t)((k * CPR + ((col >> 3) ^ swz(k))) * 16 + ((col >> 2) & 1) * 8);
            }
        }
    }
    __device__ inline void issue(int kt, uint32_t tile) const {
        const char* b = base + (int64_t)kt * kstep;
        const int wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            dma16(b, voff[i], __builtin_amdgcn_readfirstlane(tile + (uint32_t)(NI * wave + i) * 1024u));
    }
    __device__ inline uint4 frag(const unsigned char* tile, int blk, int ks) const {
        if (KIND == SRC_KCONTIG) {
            return *reinterpret_cast<const uint4*>(tile + (roff[blk] ^ (uint32_t)(ks * 32)));
        } else {
            typedef __attribute__((address_space(3))) short4_t lds_s4;
            const uint32_t o = roff[blk] + ks * (16 * CPR * 16);
            const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(tile + o));
            const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(tile + o + 4 * CPR * 16));
            uint2 a = __builtin_bit_cast(uint2, lo), b2 = __builtin_bit_cast(uint2, hi);
            return make_uint4(a.x, a.y, b2.x, b2.y);
        }
    }
};

// Epilogue of a 128 x 64 wave tile.  `lds_free` is LDS no load is in flight to (4 KB per wave) for the
// staged stores; `red` (64 floats per wave) takes the column sums and is the space of the bias slices, which
// an epilogue with column sums does not use.
template <class Epi, int MB, int TN>
__device__ inline void tile_epilogue(const Epi& epi, float16_t (&acc)[MB][2], unsigned char* lds_free,
                                     const float* lds_bias, float* red, const uint4 (&first)[4], int p, int tm,
                                     int tiles_m, int r0, int c0, int rows, int cols, int wm, int wn) {
    static_assert(!(Epi::kBias && Epi::kColSum), "the bias slice and the column sums share LDS");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 31, lg = lane >> 5;
    float cs[Epi::kColSum ? 32 : 1];
    // staged stores: a per-wave patch of 32 rows x 128 bytes whose 16-byte chunks are XOR-swizzled by the
    // row, written by the lanes that own the values and read back as whole 128-byte row segments
    unsigned char* patch = lds_free + wave * 4096;
    uint4 cur[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) cur[o] = first[o];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int r = r0 + wm + 32 * i + lr;
        const int rc = r < rows ? r : rows - 1;
        if (Epi::kStagePers) {
            static_assert(!Epi::kStagePers || Epi::kES == 2, "staged stores are for 2-byte outputs");
            uint4 second[4];
            uint4 nxt[4];
            if constexpr (Epi::kPrefetch) {  // operands of block i + 1 are requested before block i is worked on
                if (i + 1 < MB) {
                    const int rn = r0 + wm + 32 * (i + 1) + lr, rnc = rn < rows ? rn : rows - 1;
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const int c = c0 + wn + 16 * o + 8 * lg;
                        nxt[o] = epi.fetch(rnc, c < cols ? c : 0);
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const int j = o >> 1, h = o & 1;
                const int c = c0 + wn + 32 * j + 16 * h + 8 * lg;
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = acc[i][j][8 * h + u];
                typename Epi::Out out;
                if constexpr (Epi::kBias) {
                    // lds_bias holds the bias of the tile's columns (clamped at the matrix edge)
                    const float4 b0 = *reinterpret_cast<const float4*>(lds_bias + wn + 32 * j + 16 * h + 8 * lg);
                    const float4 b1 = *reinterpret_cast<const float4*>(lds_bias + wn + 32 * j + 16 * h + 8 * lg + 4);
                    v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w;
                    v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
                    epi.compute_biased(v, out);
                } else if constexpr (Epi::kPrefetch) {
                    epi.compute_fetched(cur[o], v, out);
                } else {
                    epi.compute(rc, c < cols ? c : 0, 8, v, out);
                }
                if (Epi::kColSum) {
                    const bool ok = (r < rows) && (c < cols);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int t = Epi::kColSum ? (8 * o + u) : 0;
                        cs[t] = (i == 0 ? 0.f : cs[t]) + (ok ? v[u] : 0.f);
                    }
                }
                const int cch = 4 * j + 2 * h + lg;
                *reinterpret_cast<uint4*>(patch + lr * 128 + ((cch ^ (lr & 7)) * 16)) = Epi::pk(out, 0).lo;
                if (Epi::kArrays == 2) second[o] = Epi::pk(out, 1).lo;
            }
#pragma unroll
            for (int a = 0; a < Epi::kArrays; ++a) {
                if (a == 1) {
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const int cch = 4 * (o >> 1) + 2 * (o & 1) + lg;
                        *reinterpret_cast<uint4*>(patch + lr * 128 + ((cch ^ (lr & 7)) * 16)) = second[o];
                    }
                }
                __builtin_amdgcn_wave_barrier();
                char* base = epi.arr(a);
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int q = it * 64 + lane, prow = q >> 3, pc = q & 7;
                    const uint4 u = *reinterpret_cast<const uint4*>(patch + prow * 128 + ((pc ^ (prow & 7)) * 16));
                    const int gr = r0 + wm + 32 * i + prow, gc = c0 + wn + pc * 8;
                    if (gr < rows && gc < cols) *reinterpret_cast<uint4*>(base + ((int64_t)gr * epi.ld + gc) * 2) = u;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if constexpr (Epi::kPrefetch) {
#pragma unroll
                for (int o = 0; o < 4; ++o) cur[o] = nxt[o];
            }
        } else {
            // `first` holds the prefetched operands of block 0 (four octets per lane); those of block
            // i + 1 are requested before block i is worked on
            uint4 nxt[4];
            if constexpr (Epi::kPrefetch) {
                if (i + 1 < MB) {
                    const int rn = r0 + wm + 32 * (i + 1) + lr, rnc = rn < rows ? rn : rows - 1;
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const int c = c0 + wn + 16 * o + 8 * lg;
                        nxt[o] = epi.fetch(rnc, c < cols ? c : 0);
                    }
                }
            }
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                typename Epi::Out outs[2];
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int c = c0 + wn + 32 * jb + 16 * o + 8 * lg;
                    float v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = acc[i][jb][8 * o + u];
                    const bool ok = (r < rows) && (c < cols);
                    if constexpr (Epi::kPrefetch) epi.compute_fetched(cur[2 * jb + o], v, outs[o]);
                    else epi.compute(rc, c < cols ? c : 0, 8, v, outs[o]);
                    if (Epi::kColSum) {
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const int t = Epi::kColSum ? (16 * jb + 8 * o + u) : 0;
                            cs[t] = (i == 0 ? 0.f : cs[t]) + (ok ? v[u] : 0.f);
                        }
                    }
                }
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int c = c0 + wn + 32 * jb + 16 * o + 8 * lg;
                    if (r < rows && c < cols) epi.flush(r, c, (cols - c < 8) ? (cols - c) : 8, outs[o]);
                }
            }
            if constexpr (Epi::kPrefetch) {
#pragma unroll
                for (int o = 0; o < 4; ++o) cur[o] = nxt[o];
            }
        }
    }
    if (Epi::kColSum) {
        // as in gemm_epilogue, over the 128 rows of the wave tile and then over the two waves of a column half
        fold_slots<16>(cs, lr);
        fold_slots<8>(cs, lr);
        fold_slots<4>(cs, lr);
        fold_slots<2>(cs, lr);
        fold_slots<1>(cs, lr);
        {
            const int j = lr >> 4, h = (lr >> 3) & 1, u = lr & 7;
            red[wave * 64 + 32 * j + 16 * h + 8 * lg + u] = cs[0];
        }
        __syncthreads();
        if (threadIdx.x < TN) {  // the two waves of a 64-column strip: wave ids s and s + TN / 64
            const int strip = threadIdx.x >> 6, col = threadIdx.x & 63;
            const float v = red[strip * 64 + col] + red[(TN / 64 + strip) * 64 + col];
            if (c0 + threadIdx.x < cols) epi.part[((int64_t)p * tiles_m + tm) * epi.ld + c0 + threadIdx.x] = v;
        }
    }
}

template <class Epi, int TN> constexpr bool pg_dx() { return std::is_same<Epi, EpiDx<bf16_t>>::value && TN == 256; }
template <int KA, int KB, class Epi, int TN>
__global__ __launch_bounds__(2 * TN, 2) void k_gemm_pers(GemmArgs<bf16_t, KA, KB, Epi, true, GEMM_NCH> g, int n_tiles) {
    typedef PgShape<TN> S;
    constexpr bool LINES = std::is_same<Epi, EpiDw>::value;  // fp32 results: stored as whole lines (epilogue_f32)
    constexpr bool DX = pg_dx<Epi, TN>();
    extern __shared__ __align__(16) unsigned char dlds[];
    const int wave = threadIdx.x >> 6;
    unsigned char* dx_even = dlds + S::kLds + 8 * TN + wave * 4096;
    const int wm = (wave / (TN / 64)) * 128, wn = (wave % (TN / 64)) * 64;
    const int per_p = g.tiles_m * g.tiles_n;
    int nk = 0;  // contraction steps of the current tile
    const uint32_t lbase = (uint32_t)(size_t)dlds;
    DmaTile<KA, PG_TM, 4, S::kWaves> A;
    DmaTile<KB, TN, 2, S::kWaves> B;
    A.set_lane(wm, false);
    B.set_lane(wn, !LINES);

    // tile ids of this workgroup: blockIdx.x, + gridDim.x, ...; the XCD remap keeps the tiles that the
    // workgroups of one XCD work on at the same time next to each other (same preference, same W(p))
    auto locate = [&](int vid, int& p, int& tm, int& tn) {
        const int id = xcd_remap(vid, n_tiles);
        p = id / per_p;
        tm = (id % per_p) / g.tiles_n;
        tn = id % g.tiles_n;
    };
    int bslot = 0;
    auto request = [&](int p, int tm, int tn) {  // first stages of a tile (and its bias slice)
        if constexpr (Epi::kBias) {
            bslot ^= 1;
            if (wave < TN / 64) {
                int c = tn * TN + 64 * wave + (threadIdx.x & 63);
                c = c < g.b.rows ? c : g.b.rows - 1;
                dma4(g.epi.bias + (int64_t)p * g.e0_pstride, (uint32_t)c * 4u,
                     __builtin_amdgcn_readfirstlane(lbase + S::kLds + (uint32_t)(bslot * (4 * TN) + wave * 256)));
            }
        }
        const auto grp = g.group(p);
        nk = grp.kdim / 32;
        A.set_tile(g.a_base(grp), (int)g.a.ld, g.a.rows, tm * PG_TM);
        B.set_tile(g.b_base(grp), (int)g.b.ld, g.b.rows, tn * TN);
#pragma unroll
        for (int st = 0; st < PG_NST - 1; ++st)
            if (st < nk) {
                A.issue(st, lbase + st * S::kStage);
                B.issue(st, lbase + st * S::kStage + PG_A_BYTES);
            }
    };

    int vid = blockIdx.x;
    if (vid >= n_tiles) return;
    int p, tm, tn;
    locate(vid, p, tm, tn);
    request(p, tm, tn);
    for (;;) {
        float16_t acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        uint4 first[4] = {};
        for (int kt = 0; kt < nk; ++kt) {
            // a wave has kLoads loads per stage in flight.  At the first step of a tile the stores of the
            // previous epilogue may still be counted as well, so everything is waited for.
            if (kt == 0 || kt == nk - 1) wait_vm<0>();
            else wait_vm<S::kLoads>();
            __syncthreads();  // stage kt is complete, and stage kt - 1 (or the last epilogue's patch) is free
            if constexpr (DX) {
                if (kt == nk - 1) {  // as below
                    Epi epi0 = g.epi;
                    shift_epi(epi0, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);
                    DxBlocks(epi0, tm * PG_TM + wm, tn * TN + wn, g.crows, g.ccols).request(0, dx_even);
                }
            } else if constexpr (Epi::kPrefetch) {
                // the epilogue's first block of act'(z): requested behind the tile's last operand stage, during the
                // last contraction step (after the products it cost 0.2 ms more per step of workload 5; two or four
                // steps earlier measured no better)
                if (kt == nk - 1) {
                    Epi epi0 = g.epi;
                    shift_epi(epi0, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);
                    const int r = tm * PG_TM + wm + (threadIdx.x & 31), rc = r < g.a.rows ? r : g.a.rows - 1;
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const int c = tn * TN + wn + 16 * o + 8 * ((threadIdx.x & 63) >> 5);
                        first[o] = epi0.fetch(rc, c < g.b.rows ? c : 0);
                    }
                }
            }
            if (kt + PG_NST - 1 < nk) {
                const uint32_t tile = lbase + (uint32_t)((kt + PG_NST - 1) % PG_NST) * S::kStage;
                A.issue(kt + PG_NST - 1, tile);
                B.issue(kt + PG_NST - 1, tile + PG_A_BYTES);
            }
            const unsigned char* ta = dlds + (kt % PG_NST) * S::kStage;
            const unsigned char* tb = ta + PG_A_BYTES;
            // all fragments of the stage are requested before the first product, so that one LDS latency is
            // exposed per step instead of one per pair of products
            uint4 fa[2][4], fb[2][2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[ks][j] = B.frag(tb, j, ks);
#pragma unroll
                for (int i = 0; i < 4; ++i) fa[ks][i] = A.frag(ta, i, ks);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if (LINES) Mma32<bf16_t>::run(fa[ks][i], fb[ks][j], acc[i][j]);
                        else Mma32<bf16_t>::run(fb[ks][j], fa[ks][i], acc[i][j]);  // transposed tile
                    }
            constexpr int kReads = ((KA == SRC_KCONTIG) ? 8 : 16) + ((KB == SRC_KCONTIG) ? 4 : 8);
            __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);  // LDS reads
            __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);      // MFMAs
        }
        __syncthreads();  // every wave is done with the stages
        const int pc = p, tmc = tm, tnc = tn;
        const float* lds_bias = reinterpret_cast<const float*>(dlds + S::kLds + bslot * (4 * TN));
        Epi epi = g.epi;
        shift_epi(epi, pc, g.e0_pstride, g.e1_pstride, g.e2_pstride);
        vid += gridDim.x;
        const bool more = vid < n_tiles;
        if (more) {
            locate(vid, p, tm, tn);
            request(p, tm, tn);  // stages 0 and 1; the epilogue below stages its stores in the third
        }
        if constexpr (LINES)
            epilogue_f32(epi, acc, nullptr, pc, tmc, g.tiles_m, tmc * PG_TM + wm, tnc * TN + wn, g.crows, g.ccols);
        else if constexpr (DX)
            dx_epilogue<4, 4>(epi, DxBlocks(epi, tmc * PG_TM + wm, tnc * TN + wn, g.crows, g.ccols), acc, dx_even,
                        dlds + (PG_NST - 1) * S::kStage + wave * 4096, reinterpret_cast<float*>(dlds + S::kLds),
                        more ? (nk < PG_NST - 1 ? nk : PG_NST - 1) * S::kLoads : 0, pc, tmc, g.tiles_m, tmc * PG_TM, tnc * TN, g.crows,
                        g.ccols, wm, wn);
        else
            tile_epilogue<Epi, 4, TN>(epi, acc, dlds + (PG_NST - 1) * S::kStage, lds_bias,
                                  reinterpret_cast<float*>(dlds + S::kLds), first, pc, tmc, g.tiles_m, tmc * PG_TM, tnc * TN,
                                  g.crows, g.ccols, wm, wn);
        if (!more) break;
    }
}

// ---- fp32 weight gradients on 64 x 64 tiles ------------------------------------------------------------------------
// k_grouped_gemm's products for dW where 128 x 128 tiles would multiply more padding (160 x 160 outputs: 64 blocks of 32 x 32
// on four tiles, 36 on nine small ones; 32 x 32: 16 and 4).  A wave owns one block; the contraction (whole 32-index steps)
// runs in the same order, so the sums keep their bits.  A step is sixteen contraction indices, six products' worth of work, so
// the operands of the next F32S_AHEAD steps are on their way in registers (one step ahead: 3.6 us more a launch for 10
// preferences x 1850 rows x 160 x 160), and the next step's are split beside this one's products (in front of them: the backward pass
// of those 78.4 us, 75.0 so; 16 x 6000 rows of 3 x 64 139 and 128).
#define F32S_AHEAD 4
template <class Epi>
__global__ __launch_bounds__(256) void k_gemm_f32_small(GemmArgs<float, SRC_KSTRIDED, SRC_KSTRIDED, Epi, true, GEMM_NCH> g) {
    constexpr int PITCH = gemm_pitch<float>(GEMM_NCH);
    __shared__ __align__(16) unsigned char lds[2][2][64 * PITCH];
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int per_p = g.tiles_m * g.tiles_n;
    const int p = id / per_p, tm = (id % per_p) / g.tiles_n, tn = id % g.tiles_n;
    Epi epi = g.epi;
    shift_epi(epi, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);
    const auto grp = g.group(p);
    const int r0 = tm * 64, c0 = tn * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    // a thread stages contraction indices 4 wave .. + 3 of row `lane` of either operand (rows past the end: the last one)
    const float* A = g.a_base(grp) + (int64_t)(4 * wave) * g.a.ld + (r0 + lane < g.a.rows ? r0 + lane : g.a.rows - 1);
    const float* B = g.b_base(grp) + (int64_t)(4 * wave) * g.b.ld + (c0 + lane < g.b.rows ? c0 + lane : g.b.rows - 1);
    const int nk = grp.kdim / 16;
    float ra[F32S_AHEAD][4], rb[F32S_AHEAD][4];
    auto load = [&](int slot, int kt) {  // (steps past the end: the last one again, so that as many loads are in flight in every step)
        const int64_t k0 = 16 * (int64_t)(kt < nk ? kt : nk - 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ra[slot][e] = A[(k0 + e) * g.a.ld];
            rb[slot][e] = B[(k0 + e) * g.b.ld];
        }
    };
    auto split = [&](int slot, uint2 (&pa)[3], uint2 (&pb)[3]) __attribute__((always_inline)) {
        split3(__builtin_bit_cast(uint4, make_float4(ra[slot][0], ra[slot][1], ra[slot][2], ra[slot][3])), pa);
        split3(__builtin_bit_cast(uint4, make_float4(rb[slot][0], rb[slot][1], rb[slot][2], rb[slot][3])), pb);
    };
    auto store = [&](const uint2 (&pa)[3], const uint2 (&pb)[3], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            *reinterpret_cast<uint2*>(lds[buf][0] + lane * PITCH + q * (GEMM_NCH * 8) + wave * 8) = pa[q];
            *reinterpret_cast<uint2*>(lds[buf][1] + lane * PITCH + q * (GEMM_NCH * 8) + wave * 8) = pb[q];
        }
    };
    float16_t acc[1][1], low;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] = low[e] = 0.f;
#pragma unroll
    for (int u = 0; u < F32S_AHEAD; ++u) load(u, u);
    {
        uint2 pa[3], pb[3];
        split(0, pa, pb);
        store(pa, pb, 0);
    }
    load(0, F32S_AHEAD);
    __syncthreads();
    for (int k0 = 0; k0 < nk; k0 += F32S_AHEAD) {
#pragma unroll
        for (int u = 0; u < F32S_AHEAD; ++u) {
            const int kt = k0 + u, cur = u & 1, nxt = (u + 1) % F32S_AHEAD;
            if (kt >= nk) break;
            const unsigned char* ta = lds[cur][0] + (wm + lr) * PITCH + lg * 16;
            const unsigned char* tb = lds[cur][1] + (wn + lr) * PITCH + lg * 16;
            uint4 fa[3], fb[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                fa[q] = *reinterpret_cast<const uint4*>(ta + q * 32);
                fb[q] = *reinterpret_cast<const uint4*>(tb + q * 32);
            }
            // the next step's operands are split beside this one's reads and products and written behind them
            uint2 pa[3], pb[3];
            split(nxt, pa, pb);
#pragma unroll
            for (int t = 0; t < 6; ++t) split_mma(t, fa, fb, acc[0][0], low);
            store(pa, pb, cur ^ 1);  // (its readers passed the barrier of the step before)
            load(nxt, kt + 1 + F32S_AHEAD);
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);  // LDS reads
            __builtin_amdgcn_sched_group_barrier(0x002, 24, 0);
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a product
                __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);
            }
            __syncthreads();
        }
    }
    acc[0][0] += low;
    if (any_undefined(acc[0][0])) {
        Operand<float, SRC_KSTRIDED, true, GEMM_NCH> a = g.a, b = g.b;
        a.base = g.a_base(grp); b.base = g.b_base(grp);
        a.kdim = b.kdim = grp.kdim;
        plain_products(a, b, r0 + wm + lr, c0 + wn + lr, grp.kdim, acc[0][0]);
    }
    epilogue_f32(epi, acc, nullptr, p, tm, g.tiles_m, r0 + wm, c0 + wn, g.crows, g.ccols);
}

// ---- bf16 weight gradients with few tiles: 64 x 64 outputs a workgroup --------------------------------------------
// dW of few preferences on 128 x 128 tiles leaves CUs without a workgroup, and its contraction may only be split where the
// grouping of its sums says so.  Smaller tiles keep every sum as it is.  A wave owns 32 x 32 outputs; a step of 32
// contraction indices is two products, so what bounds a workgroup is the latency of its operands: eight stages of 8 KB,
// six of them on their way, two multiplied behind one barrier (one by one: 14.4 us a launch for 24 preferences x 1250 rows x 256 x
// 256, 13.7 so; the 126 MB of operands that its workgroups request come out of the L2s at 9.2 TB/s, a third of what those give).
#define SG_NST 8
#define SG_STAGE 8192
template <class Epi>
__global__ __launch_bounds__(256) void k_gemm_small(GemmArgs<bf16_t, SRC_KSTRIDED, SRC_KSTRIDED, Epi, true, GEMM_NCH> g) {
    __shared__ __align__(16) unsigned char dlds[SG_NST * SG_STAGE];
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int per_p = g.tiles_m * g.tiles_n;
    const int p = id / per_p, tm = (id % per_p) / g.tiles_n, tn = id % g.tiles_n;
    Epi epi = g.epi;
    shift_epi(epi, p, g.e0_pstride, g.e1_pstride, g.e2_pstride);
    const int r0 = tm * 64, c0 = tn * 64;
    const int wave = threadIdx.x >> 6, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    DmaTile<SRC_KSTRIDED, 64, 1, 4> A, B;
    A.set_lane(wm, false);
    B.set_lane(wn, false);
    const auto grp = g.group(p);
    A.set_tile(g.a_base(grp), (int)g.a.ld, g.a.rows, r0);
    B.set_tile(g.b_base(grp), (int)g.b.ld, g.b.rows, c0);
    float16_t acc[1][1];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] = 0.f;
    const int nk = grp.kdim / 32;
    const uint32_t lbase = (uint32_t)(size_t)dlds;
    auto issue = [&](int kt) {
        const uint32_t tile = lbase + (uint32_t)(kt % SG_NST) * SG_STAGE;
        A.issue(kt, tile);
        B.issue(kt, tile + SG_STAGE / 2);
    };
    for (int st = 0; st < SG_NST - 2 && st < nk; ++st) issue(st);
    // two steps behind one barrier (their four products are one chain; a step by itself is barrier, LDS reads and two products one
    // after the other, 360 cycles of which the products are 64); nk odd: the last one alone
    for (int kt = 0; kt < nk; kt += 2) {
        // two loads a stage and wave; the two oldest stages are the ones multiplied next
        const int behind = nk - 2 - kt;
        if (behind >= SG_NST - 4) wait_vm<2 * (SG_NST - 4)>();
        else if (behind == 3) wait_vm<6>();
        else if (behind == 2) wait_vm<4>();
        else if (behind == 1) wait_vm<2>();
        else wait_vm<0>();
        __syncthreads();  // stages kt and kt + 1 have landed for every wave, and everyone is done with the two before
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (kt + SG_NST - 2 + u < nk) issue(kt + SG_NST - 2 + u);
        const unsigned char* ta = dlds + (kt % SG_NST) * SG_STAGE;
        const bool two = kt + 1 < nk;  // (kt is even and SG_NST too: the other stage follows in LDS)
        uint4 fa[4], fb[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            fa[ks] = A.frag(ta + (ks >> 1) * SG_STAGE, 0, ks & 1);
            fb[ks] = B.frag(ta + (ks >> 1) * SG_STAGE + SG_STAGE / 2, 0, ks & 1);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) Mma32<bf16_t>::run(fa[ks], fb[ks], acc[0][0]);
        if (two) {
#pragma unroll
            for (int ks = 2; ks < 4; ++ks) Mma32<bf16_t>::run(fa[ks], fb[ks], acc[0][0]);
        }
    }
    epilogue_f32(epi, acc, nullptr, p, tm, g.tiles_m, r0 + wm, c0 + wn, g.crows, g.ccols);
}

// ---- fused forward: observations -> every hidden layer -> output layer (bf16, width 512 or 256) -------
// (paper Sec. III-C: the target network of a preference applied to that preference's environments, in the
// rollout and in the update.)  One workgroup of W / 64 waves carries 128 rows of one preference through the
// whole network, tile after tile (width 512: eight waves, one workgroup per CU; width 256: four waves and half the
// tile, two per CU).  The activations of the tile live in LDS (128 rows x 2 W bytes, 16-byte chunks XOR-swizzled by
// the row) and are rewritten in place layer after layer; HBM sees the observations once, the outputs once
// and, in the saving variant, the stores of h and act'(z) that the backward pass reads -- never a load of
// an activation.
// Wave w owns output features [64 w, 64 w + 64) of every layer for all 128 rows: its slice of W_l(p) is
// used by no other wave, so the W fragments go from global memory (they sit in L2: 64 tiles share one
// W(p)) straight into registers, half a super-step at a time ("unit": 16 products, 32 contraction indices
// per lane group).  The kernel reads them from a copy of the matrices in fragment order
// (k_theta_fragment_order, made by the same call): every load instruction then covers 1 KB of consecutive
// addresses.  Read from the row-major matrices the same stream takes 32 bytes from each of 32 rows per
// instruction, and the workgroups of a CU, 64 KB of such lines in flight against its vector cache, fetch
// lines from L2 more than once: streamed alone, without the products, W moved at 9.7 TB/s row-major and
// 15.3 TB/s in fragment order, and a launch of workload 5 spends most of its time on exactly this stream.
// Inside a super-step lane group g
// of product jj covers contraction indices 64 s + 32 g + 8 jj .. + 8 for both operands.  The bias enters
// as the initial value of the accumulators.  A layer ends with a barrier, the epilogue (activation, its
// derivative, the in-place rewrite of the tile, the stores of the saving variant) and a second barrier;
// the products and the epilogue of a workgroup do not overlap, and with 128 KB of LDS for the tile there is
// one workgroup per CU.  Measured on workload 5 the time of a launch splits, additively, into the W
// requests, the products, the epilogue arithmetic and a fixed part per tile (observation gather, first
// requests, barriers).
#define FF_ROWS 128

struct FusedFwdArgs {
    const float* x;           // observations, time-major rows of O values
    bf16_t* x0;               // saving, optional: receives the gathered observations, compact [P][Mp][ldx] bf16
    const bf16_t* theta_mat;  // [P][mat_len]: the output layer's matrix is read from here
    const bf16_t* theta_frag; // [P][mat_len]: the first and the hidden layers' matrices in fragment order
    const float* theta_vec;   // [P][vec_len]
    int64_t mat_len, vec_len;
    int64_t mat_off[MORLAX_MAX_LAYERS], vec_off[MORLAX_MAX_LAYERS];
    int64_t frag_len, frag_off[MORLAX_MAX_LAYERS];  // the fragment-order copy: elements per preference, layer starts
    int32_t Opad;  // O rounded up to a multiple of 64: the first layer's contraction, zero-filled beyond O
    bf16_t* H;    // saving: h of layer l at H + l * lstride; else the last layer's h only
    gfix16_t* G;  // saving: act'(z) of layer l at G + l * lstride
    int64_t lstride;
    int32_t L, O, M, tiles_m, n_tiles;
    int32_t Mp, ldx;  // saving: rows per preference of H, G and x0 (copies of row M - 1 beyond M), row length of x0
    // output layer (applied to the tile's last hidden activations while they are still in LDS)
    int64_t head_mat_off, head_vec_off, logsig_off;
    int32_t out_dim, tanh_cols;  // leading output columns that are squashed by tanh (the actor's means)
    int32_t adim, sig_state;     // action width; 1: log sigma = output columns [adim, 2 adim) of the same row
    RowMap rm;
    float* out;        // time-major [.., N, out_dim]
    float* saved_out;  // saving: compact [P][M][OUT_PITCH]
    const float* eps;  // actor with sampling: noise, and the two outputs below
    float* act;
    float* logp;
};

// Fragment order of a [W][K] bf16 matrix (K a multiple of 64): the 16-byte pieces of W in the order in
// which the fused forward requests them, so that each of its load instructions reads 1 KB of consecutive
// addresses (eight whole cache lines) instead of 32 bytes from each of 32 rows.  Wave v of the forward owns
// output features [64 v, 64 v + 64); its stream is K / 32 units of 4 KB; unit u holds four 1 KB blocks
// (j, e), j = feature half, e = which 16 bytes; lane (lg, lr) of a block holds, for feature
// 64 v + 32 j + swap_bits23(lr), the contraction indices 64 (u / 2) + 32 lg + 16 (u % 2) + 8 e + [0, 8).
// One workgroup moves a super-step pair of units of one j: 32 rows x 128 bytes, whole lines in and out.
struct FragOrderArgs {
    const bf16_t* src;  // [P][mat_len] row-major matrices
    bf16_t* dst;        // [P][frag_len]
    int64_t mat_len, frag_len;
    int64_t mat_off[MORLAX_MAX_LAYERS], frag_off[MORLAX_MAX_LAYERS];
    int32_t K[MORLAX_MAX_LAYERS];     // contraction length in the copy (a multiple of 64)
    int32_t Ksrc[MORLAX_MAX_LAYERS];  // columns of the row-major matrix; the copy is zero beyond them
    int32_t g0[MORLAX_MAX_LAYERS + 1];  // first workgroup of layer l; g0[L] = workgroups per preference
    int32_t L;
};

__global__ __launch_bounds__(256) void k_theta_fragment_order(FragOrderArgs a) {
    const int p = blockIdx.y;
    int l = 0;
    while (l + 1 < a.L && (int)blockIdx.x >= a.g0[l + 1]) ++l;
    const int K = a.K[l], g = blockIdx.x - a.g0[l];
    const int per_wave = 2 * (K >> 6);
    const int v = g / per_wave, r = g % per_wave, sstep = r >> 1, j = r & 1;
    const int wq = threadIdx.x >> 6, ln = threadIdx.x & 63, ub = wq >> 1, e = wq & 1, lg = ln >> 5, lr = ln & 31;
    const int u = 2 * sstep + ub;
    const bf16_t* Wsrc = a.src + (int64_t)p * a.mat_len + a.mat_off[l];
    char* D = reinterpret_cast<char*>(a.dst + (int64_t)p * a.frag_len + a.frag_off[l]);
    const int f = 64 * v + 32 * j + swap_bits23(lr);
    const int k0 = (sstep * 128 + ub * 32 + lg * 64 + e * 16) >> 1, Ks = a.Ksrc[l];
    uint4 q;
    if (Ks == K) {
        q = *reinterpret_cast<const uint4*>(Wsrc + (int64_t)f * K + k0);
    } else {  // an observation width that is no multiple of 64: element by element, zeros beyond it
        const unsigned short* row = reinterpret_cast<const unsigned short*>(Wsrc) + (int64_t)f * Ks;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = (k0 + 2 * i < Ks) ? row[k0 + 2 * i] : 0u, hi = (k0 + 2 * i + 1 < Ks) ? row[k0 + 2 * i + 1] : 0u;
            w[i] = lo | (hi << 16);
        }
        q = make_uint4(w[0], w[1], w[2], w[3]);
    }
    *reinterpret_cast<uint4*>(D + (int64_t)v * (K >> 5) * 4096 + u * 4096 + j * 2048 + e * 1024 + ln * 16) = q;
}

template <int ACT, bool SAVE, int WD>
__global__ __launch_bounds__(WD, 2) void k_mlp_fused_fwd(FusedFwdArgs a) {
    constexpr int RB = 2 * WD;           // bytes of a tile row
    constexpr int NW = WD / 64;          // waves: 64 output features each
    constexpr int TILE_BYTES = FF_ROWS * RB;
    extern __shared__ __align__(16) unsigned char dlds[];
    // One workgroup per CU walks the tiles (no launch gap, no register spill in the saving variant).  Everything
    // derived from the lane is formed again for every tile behind opaque(): kept across tiles it would occupy
    // registers that the products and the epilogue need.
    for (int vt = blockIdx.x; vt < a.n_tiles; vt += gridDim.x) {
        const int lane = opaque((int)(threadIdx.x & 63)), lr = lane & 31, lg = lane >> 5;
        const int wave = __builtin_amdgcn_readfirstlane(opaque((int)(threadIdx.x >> 6)));
        const int tile = xcd_remap(vt, a.n_tiles);
        const int p = tile / a.tiles_m, m0 = (tile % a.tiles_m) * FF_ROWS;
        const int rows = a.M - m0 < FF_ROWS ? a.M - m0 : FF_ROWS;
        const int srows = SAVE ? a.Mp - m0 : 0;  // rows to save
        const int wn = wave * 64;

        const bf16_t* Wp = a.theta_frag + (int64_t)p * a.frag_len;
        const float* bp = a.theta_vec + (int64_t)p * a.vec_len;
        // the wave's stream of W_l(p) in fragment order: a uniform base and the lane's 16 bytes
        auto w_stream = [&](int l) {
            const int K = l == 0 ? a.Opad : WD;
            return reinterpret_cast<const char*>(Wp + a.frag_off[l]) + (int64_t)wave * (K >> 5) * 4096;
        };
        // unit u of a layer = 32 contraction indices per lane group, 4 KB of the wave's stream (fragment order)
        auto load_w = [&](u32x4_t (&wf)[2][2], const char* w, int u) __attribute__((always_inline)) {
            const uint32_t lo = (uint32_t)lane * 16u;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) wf[j][e] = *reinterpret_cast<const u32x4_t*>(w + u * 4096 + (j * 2048 + e * 1024) + lo);
        };
        // W fragments: a ring of four buffers.  In the hidden layers a unit is requested three units ahead of its use: the
        // stores of the saving variant raise the latency of a W request from 140 to 750 cycles on average, a unit's
        // products take 1000.  Only a layer's first unit is requested ahead of the epilogue in front of it, whose registers
        // the other buffers are.  (128 preferences x 2048 rows of 4 x 512, with the fragment-order copy: 856 -> 835 us.)
        u32x4_t wfa[2][2], wfb[2][2], wfc[2][2], wfd[2][2];
        float16_t acc[4][2];
        const char* wp = w_stream(0);

        {  // the tile's observations, gathered from the time-major tensor and rounded to bf16; rows past the end
           // repeat the last row (saved up to Mp, no output).  The saving variant keeps the compact copy that the first
           // layer's dW product reads.  2^sh pieces of eight values a row, requested G a thread at a time (one by one, each
           // with two divisions: 13 thousand of the 110 thousand cycles of a tile of 3 x 256 with 11 observations; us, 32 preferences x
           // 8192 rows of it 121 -> 115, saving 242 -> 237; 64 x 2048 of 2 x 256 with 100 71 -> 57, 114 -> 110).
            constexpr int G = 4 * 256 / WD;
            const int O = a.O, np = a.Opad >> 3, sh = 32 - __builtin_clz(np - 1), n_id = FF_ROWS << sh;
            auto obs_row = [&](int r) __attribute__((always_inline)) {
                return a.x + (uint32_t)a.rm.row(p, m0 + (r < rows ? r : rows - 1)) * (uint32_t)O;  // (the tensor stays below 4 GiB)
            };
            auto put_piece = [&](const float (&v)[8], int r, int c) __attribute__((always_inline)) {
                const uint4 q = pack_chunk<bf16_t>(v);
                *reinterpret_cast<uint4*>(dlds + r * RB + ((c ^ (r & 15)) * 16)) = q;
                if (SAVE && a.x0 && r < srows && 8 * c < a.ldx)
                    *reinterpret_cast<uint4*>(a.x0 + ((int64_t)p * a.Mp + m0 + r) * a.ldx + 8 * c) = q;
            };
            if (O >= 8) {
                for (int first = opaque((int)threadIdx.x); first < n_id; first += G * WD) {  // (n_id: a multiple of G WD)
                    u32x4_t q[G][2];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const int id = first + g * WD;
                        obs_get(q[g], obs_row(id >> sh), id & ((1 << sh) - 1), O);
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const int id = first + g * WD, c = id & ((1 << sh) - 1);
                        float v[8];
                        obs_place(v, q[g], c, O);
                        if (c < np) put_piece(v, id >> sh, c);
                    }
                }
            } else {  // rows shorter than a piece, element by element; the zeros behind them by all threads
                for (int r = threadIdx.x; r < FF_ROWS; r += WD) {
                    const float* row = obs_row(r);
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = e < O ? row[e < O ? e : O - 1] : 0.f;
                    put_piece(v, r, 0);
                }
                for (int id = opaque((int)threadIdx.x) + FF_ROWS; id < FF_ROWS * np; id += WD) {
                    const float zero[8] = {};
                    put_piece(zero, id % FF_ROWS, id / FF_ROWS);
                }
            }
        }
        load_w(wfa, wp, 0);
        // fragment addresses: row 32 i + lr, chunk (8 s + 4 lg + jj) ^ (lr & 15)
        const int x = lr & 15;
        const unsigned char* arow = dlds + lr * RB;
        uint32_t aoff[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) aoff[jj] = (uint32_t)(((4 * lg + jj) ^ (x & 7)) * 16);
        const int sflip = x >> 3;

        // one unit: 16 products; HALF = u & 1 picks the chunks 2 HALF, 2 HALF + 1 of the super-step
        auto unit = [&](const u32x4_t (&wf)[2][2], int u, auto half_tag) __attribute__((always_inline)) {
            constexpr int HALF = decltype(half_tag)::value;
            const unsigned char* as = arow + ((u >> 1) ^ sflip) * 128;
            uint4 fa[2][4];
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int i = 0; i < 4; ++i) fa[jj][i] = *reinterpret_cast<const uint4*>(as + i * (32 * RB) + aoff[2 * HALF + jj]);
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) Mma32<bf16_t>::run(__builtin_bit_cast(uint4, wf[j][jj]), fa[jj][i], acc[i][j]);
        };
        // lane n of `bias` holds b_l[wn + n]; every accumulator of a lane's octet o starts from its feature's bias
        auto init_acc = [&](float bias) __attribute__((always_inline)) {
            const int at = (opaque(lane) >> 5) * 32;  // (formed here: addresses held across the epilogue would spill)
#pragma unroll
            for (int o = 0; o < 4; ++o)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float b = __int_as_float(__builtin_amdgcn_ds_bpermute(at + 4 * (16 * o + u), __float_as_int(bias)));
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i][o >> 1][8 * (o & 1) + u] = b;
                }
        };
        auto load_bias = [&](int l) { return bp[a.vec_off[l] + wn + lane]; };

        init_acc(load_bias(0));
        __syncthreads();
        constexpr std::integral_constant<int, 0> even{};
        constexpr std::integral_constant<int, 1> odd{};
        auto step = [&](u32x4_t (&next)[2][2], const char* w, int un, const u32x4_t (&wf)[2][2], int u, auto half) __attribute__((always_inline)) {
            load_w(next, w, un);
            __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the products they overlap with
            unit(wf, u, half);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto finish = [&](int l, bool more) __attribute__((always_inline)) {
            __syncthreads();  // every wave has read the layer's input for the last time
            const float bnext = load_bias(more ? l + 1 : l);
            {
                const int ol = opaque(lane), olr = ol & 31, olg = ol >> 5, ox = ol & 15;
                unsigned char* hrow = dlds + olr * RB;
                unsigned char* patch = dlds + TILE_BYTES + wave * 4096;
                gfix16_t* Gl = SAVE ? a.G + (int64_t)l * a.lstride + ((int64_t)p * a.Mp + m0) * WD + wn : nullptr;
                bf16_t* Hl = SAVE ? a.H + (int64_t)l * a.lstride + ((int64_t)p * a.Mp + m0) * WD + wn : nullptr;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint4 gq[4], hq[4];
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const int j = o >> 1, h = o & 1;
                        float v[8], g[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) act_pair<bf16_t, ACT, true>(acc[i][j][8 * h + u], v[u], g[u]);
                        const int cc = 8 * wave + 4 * j + 2 * h + olg;
                        hq[o] = pack_chunk<bf16_t>(v);
                        *reinterpret_cast<uint4*>(hrow + i * (32 * RB) + ((cc ^ ox) * 16)) = hq[o];
                        if (SAVE) gq[o] = pack8(g, (const gfix16_t*)nullptr).lo;
                    }
                    // act'(z) and h leave through the wave's patch as whole 128-byte row segments, row block by row
                    // block between the epilogue's arithmetic (h read back from the tile after the closing barrier and
                    // stored as whole rows cost 1 ms more per step of workload 5: those stores sat in front of the
                    // next layer's first requests)
                    if (SAVE) {
#pragma unroll
                        for (int arr = 0; arr < 2; ++arr) {
#pragma unroll
                            for (int o = 0; o < 4; ++o) {
                                const int cch = 4 * (o >> 1) + 2 * (o & 1) + olg;
                                *reinterpret_cast<uint4*>(patch + olr * 128 + ((cch ^ (olr & 7)) * 16)) = arr ? hq[o] : gq[o];
                            }
                            __builtin_amdgcn_wave_barrier();
                            char* dst = arr ? reinterpret_cast<char*>(Hl) : reinterpret_cast<char*>(Gl);
#pragma unroll
                            for (int it = 0; it < 4; ++it) {
                                const int prow = it * 8 + (ol >> 3), pc = ol & 7;
                                const uint4 u = *reinterpret_cast<const uint4*>(patch + prow * 128 + ((pc ^ (prow & 7)) * 16));
                                const int gr = 32 * i + prow;
                                // (a guard per store although whole row blocks are saved or not: the blocks it makes keep
                                // the compiler from mixing row blocks, which spills)
                                if (gr < srows) *reinterpret_cast<uint4*>(dst + ((int64_t)gr * WD + pc * 8) * 2) = u;
                            }
                            __builtin_amdgcn_wave_barrier();
                        }
                    }
                }
            }
            if (more) {
                __syncthreads();  // the layer's output is complete in LDS
                init_acc(bnext);
            }
        };
        const char* wq = w_stream(a.L > 1 ? 1 : 0);
        const int nU = a.Opad >> 5;
        for (int u = 0; u < nU; u += 2) {
            const bool last = u + 2 == nU;
            step(wfb, wp, u + 1, wfa, u, even);
            step(wfa, last ? wq : wp, last ? 0 : u + 2, wfb, u + 1, odd);
        }
        finish(0, a.L > 1);
        for (int l = 1; l < a.L; ++l) {
            const bool more = l + 1 < a.L;
            wp = wq;
            wq = w_stream(more ? l + 1 : l);
            constexpr int NU = WD / 32;
            load_w(wfb, wp, 1);
            load_w(wfc, wp, 2);
            for (int u = 0; u < NU - 4; u += 4) {
                step(wfd, wp, u + 3, wfa, u, even);
                step(wfa, wp, u + 4, wfb, u + 1, odd);
                step(wfb, wp, u + 5, wfc, u + 2, even);
                step(wfc, wp, u + 6, wfd, u + 3, odd);
            }
            step(wfd, wp, NU - 1, wfa, NU - 4, even);
            step(wfa, wq, 0, wfb, NU - 3, odd);
            unit(wfc, NU - 2, even);
            __builtin_amdgcn_sched_barrier(0);
            unit(wfd, NU - 1, odd);
            finish(l, more);
        }

        // output layer: wave w takes rows 16 w .. 16 w + 15 of the tile with 16x16x32 products; lane (hl, hg)
        // supplies row hl / output hl at contraction chunk 4 u + hg and receives output hl of rows 4 hg + e
        // (width 256: four waves, two passes of 64 rows).  Its weights, biases and noise are requested ahead of the barrier
        // that completes the last hidden layer: behind it they were three round trips to memory one after the other.
        const int hl = lane & 15, hg = lane >> 4;
        const bool b_ok = hl < a.out_dim;
        const bool a_ok = hl < a.adim;  // lanes that hold an action mean
        u32x4_t fb[WD / 32];
        {
            const bf16_t* wrow = a.theta_mat + (int64_t)p * a.mat_len + a.head_mat_off + (int64_t)(b_ok ? hl : 0) * WD;
#pragma unroll
            for (int u = 0; u < WD / 32; ++u) fb[u] = *reinterpret_cast<const u32x4_t*>(wrow + 8 * (4 * u + hg));
        }
        const float hbias = bp[a.head_vec_off + (b_ok ? hl : 0)];
        float ls_p = 0.f;
        if (a.eps && a_ok && !a.sig_state) ls_p = bp[a.logsig_off + hl];
        float noise[8 / NW][4];
        int64_t orow[8 / NW][4];
#pragma unroll
        for (int pass = 0; pass < 8 / NW; ++pass)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tr = 16 * (wave + NW * pass) + 4 * hg + e;
                orow[pass][e] = a.rm.row(p, m0 + (tr < rows ? tr : 0));
                noise[pass][e] = 0.f;
                if (a.eps && a_ok && tr < rows) noise[pass][e] = a.eps[orow[pass][e] * a.adim + hl];
            }
        __syncthreads();  // the last hidden layer's output is complete in LDS
#pragma unroll
        for (int pass = 0; pass < 8 / NW; ++pass) {
            const int wv = wave + NW * pass;
            const int r = 16 * wv + hl;
            const unsigned char* hrow = dlds + r * RB;
            float4_t c = {0.f, 0.f, 0.f, 0.f}, c2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < WD / 32; u += 2) {
                const uint4 f0 = *reinterpret_cast<const uint4*>(hrow + (((4 * u + hg) ^ (r & 15)) * 16));
                const uint4 f1 = *reinterpret_cast<const uint4*>(hrow + (((4 * u + 4 + hg) ^ (r & 15)) * 16));
                Mma16<bf16_t>::run(f0, __builtin_bit_cast(uint4, fb[u]), c);
                Mma16<bf16_t>::run(f1, __builtin_bit_cast(uint4, fb[u + 1]), c2);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] += c2[e];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tr = 16 * wv + 4 * hg + e, m = m0 + tr;
                const bool ok = (tr < rows) && b_ok;
                const float z = c[e] + hbias;
                const float o = (hl < a.tanh_cols) ? tanhf(z) : z;
                const int64_t row = orow[pass][e];
                float term = 0.f;
                // a state-dependent log sigma sits adim columns to the right, in the same group of 16 lanes
                const float ls_s = __shfl(o, (lane & 48) | ((hl + a.adim) & 15), 64);
                if (ok) {
                    a.out[row * a.out_dim + hl] = o;
                    if (SAVE) a.saved_out[((int64_t)p * a.M + m) * OUT_PITCH + hl] = o;
                    if (a.eps && a_ok) {
                        const float ls = a.sig_state ? ls_s : ls_p;
                        const float ep = noise[pass][e];
                        a.act[row * a.adim + hl] = o + expf(ls) * ep;
                        term = -0.5f * ep * ep - ls;
                    }
                }
                if (a.eps) {
                    term += __shfl_xor(term, 8, 64);
                    term += __shfl_xor(term, 4, 64);
                    term += __shfl_xor(term, 2, 64);
                    term += __shfl_xor(term, 1, 64);
                    if (tr < rows && hl == 0) a.logp[row] = term - 0.918938533204672742f * (float)a.adim;
                }
            }
        }
        __syncthreads();  // the tile's last readers are done before the next tile is written
    }
}

// ---- optional event timing of the GEMM launches ------------------------------------------------
#include <vector>
struct GemmProf {
    struct Rec { hipEvent_t a, b; int kind; double flops; };
    std::vector<Rec> recs;
    size_t used = 0;
    bool on = false;
};

int prof_begin(morlax_ctx* c) {
    if (!c->prof) c->prof = new GemmProf;
    c->prof->used = 0;
    c->prof->on = true;
    return 0;
}

void prof_free(morlax_ctx* c) {
    if (!c->prof) return;
    for (auto& r : c->prof->recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    delete c->prof;
    c->prof = nullptr;
}

int prof_end(morlax_ctx* c, double* ms, int64_t* launches, double* flops) {
    GemmProf* pr = c->prof;
    pr->on = false;
    for (int k = 0; k < MORLAX_GEMM_KINDS; ++k) { ms[k] = 0.0; launches[k] = 0; flops[k] = 0.0; }
    if (pr->used == 0) return 0;
    for (size_t i = 0; i < pr->used; ++i) {
        float t = 0.f;
        if (hipEventSynchronize(pr->recs[i].b) != hipSuccess) return -1;  // (launches may be spread over streams)
        if (hipEventElapsedTime(&t, pr->recs[i].a, pr->recs[i].b) != hipSuccess) return -1;
        ms[pr->recs[i].kind] += t;
        launches[pr->recs[i].kind] += 1;
        flops[pr->recs[i].kind] += pr->recs[i].flops;
    }
    pr->used = 0;
    return 0;
}

static GemmProf::Rec* prof_take(const morlax_ctx* c, int kind, double flops) {
    GemmProf* pr = c->prof;
    if (!pr || !pr->on) return nullptr;
    if (pr->used == pr->recs.size()) {
        GemmProf::Rec r;
        if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return nullptr;
        pr->recs.push_back(r);
    }
    GemmProf::Rec* r = &pr->recs[pr->used++];
    r->kind = kind;
    r->flops = flops;
    return r;
}

// The direct-to-LDS kernel serves bf16 GEMMs of compact operands whose contraction length is a multiple
// of 32 and whose addresses are 16-byte aligned; everything else runs k_grouped_gemm.
template <int KIND>
static bool dma_operand_ok(const void* base, int64_t ld, int rows, int kdim, int64_t pstride) {
    if ((reinterpret_cast<uintptr_t>(base) & 15) || (ld & 7) || (pstride & 7)) return false;
    if (KIND == SRC_KCONTIG) return rows >= 1 && (int64_t)rows * ld * 2 < (int64_t(1) << 31);
    return rows >= 8 && (rows & 7) == 0 && (64 * ld + rows) * 2 < (int64_t(1) << 31);
}
static int resident_slots() {  // workgroups of the persistent kernel: two per CU
    static int n = 0;
    if (n == 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        n = 2 * cus;
    }
    return n;
}

template <typename T, int KA, int KB, class Epi, bool FAST, int NCH>
static bool launch_special(GemmArgs<T, KA, KB, Epi, FAST, NCH>& g, int P, int nb, hipStream_t s) {
    if constexpr (std::is_same<T, bf16_t>::value && FAST && (KA == SRC_KCONTIG || KA == SRC_KSTRIDED) &&
                  (KB == SRC_KCONTIG || KB == SRC_KSTRIDED)) {
        if (g.a.kdim < 32 || (g.a.kdim & 31)) return false;
        if (!dma_operand_ok<KA>(g.a.base, g.a.ld, g.a.rows, g.a.kdim, g.a_pstride)) return false;
        if (!dma_operand_ok<KB>(g.b.base, g.b.ld, g.b.rows, g.b.kdim, g.b_pstride)) return false;
        // large problems: persistent kernel, 256 x 256 tiles (one workgroup of eight waves per CU) when the
        // output is at least that wide and there is a tile for every CU, else 256 x 128 tiles (two workgroups
        // of four waves per CU) as soon as those fill the resident workgroups
        const int ptm = (g.crows + PG_TM - 1) / PG_TM;
        auto launch_pers = [&](auto tn_tag, int slots) {
            constexpr int TN = decltype(tn_tag)::value;
            const int ptn = (g.ccols + TN - 1) / TN, pnt = ptm * ptn * P;
            static bool pattr_set = false;
            constexpr int plds = PgShape<TN>::kLds + 8 * TN + (pg_dx<Epi, TN>() ? PgShape<TN>::kWaves * 4096 : 0);
            if (!pattr_set) {
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_pers<KA, KB, Epi, TN>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, plds);
                pattr_set = true;
            }
            g.tiles_m = ptm;
            g.tiles_n = ptn;
            const int grid = pnt < slots ? pnt : slots;
            k_gemm_pers<KA, KB, Epi, TN><<<grid, 2 * TN, plds, s>>>(g, pnt);
        };
        if (g.crows >= 64) {
            const int slots = resident_slots();
            // (the wide shape as soon as there is a tile per CU: a third fewer operand bytes per product through the
            // vector cache, whose requests in flight are what the products wait for; dW at W = 512 with two tiles per
            // workgroup: 8.3 -> 7.9 ms per step of workload 5, with one tile per workgroup at workload 4: 0.945 -> 0.915)
            if (g.ccols >= 256 && ptm * ((g.ccols + 255) / 256) * P >= slots / 2) {
                launch_pers(std::integral_constant<int, 256>{}, slots / 2);
                return true;
            }
            if (ptm * ((g.ccols + 127) / 128) * P >= slots) {
                launch_pers(std::integral_constant<int, 128>{}, slots);
                return true;
            }
        }
        if constexpr (std::is_same<Epi, EpiDw>::value) {
            // fewer 128 x 128 tiles than CUs, and no more 64 x 64 ones than run at once (two per CU, by their LDS): beyond that
            // the operands read twice as often cost more than the idle CUs.  us, large and small, by preferences x rows x 256 x
            // 256: 24 x 1250 (384 small tiles) 19 and 14, 20 x 2369 (320) 29 and 19, 24 x 4531 (384) 51 and 49; 40 x 5786
            // (640) 67 and 89, 60 x 789 (960) 18 and 20, 60 x 6838 104 and 144
            const int stm = (g.crows + 63) / 64, stn = (g.ccols + 63) / 64;
            if (nb < resident_slots() / 2 && stm * stn > g.tiles_m * g.tiles_n && (int64_t)stm * stn * P <= resident_slots()) {
                g.tiles_m = stm;
                g.tiles_n = stn;
                k_gemm_small<Epi><<<stm * stn * P, 256, 0, s>>>(g);
                return true;
            }
        }
        static bool attr_set = false;
        constexpr int lds_bytes = DMA_NST * DMA_STAGE_BYTES;
        if (!attr_set) {
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dma<KA, KB, Epi>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            attr_set = true;
        }
        k_gemm_dma<KA, KB, Epi><<<nb, 256, lds_bytes, s>>>(g);
        return true;
    } else if constexpr (std::is_same<T, float>::value && std::is_same<Epi, EpiDw>::value) {
        // fewer blocks of 32 x 32 to multiply, and fewer rounds of a workgroup per CU by the factor that a round is shorter:
        // four times less work, but every operand is read twice as often.  Rounds, and us on large and on small tiles: 2 and 5
        // 46 and 27 (10 preferences x 1850 rows x 160 x 160), 4 and 15 181 and 164 (6 x 512 x 1568 x 1568), 2 and 7 46 and 45 to
        // 48 (4096 rows in all x 416 x 416), 3 and 12 125 and 133 (3 x 512 x 1952 x 1952), 9 and 34 344 and 356 (16 x 512 x
        // 1440 x 1440), 2 and 8 559 and 652 (2 x 4096 x 1952 x 1952).
        const int stm = (g.crows + 63) / 64, stn = (g.ccols + 63) / 64, cus = resident_slots() / 2;
        auto rounds = [&](int64_t tiles) { return (tiles * P + cus - 1) / cus; };
        if (stm * stn >= 4 * g.tiles_m * g.tiles_n || (g.a.kdim & 31)) return false;
        if (4 * rounds(stm * stn) > 15 * rounds(g.tiles_m * g.tiles_n)) return false;
        g.tiles_m = stm;
        g.tiles_n = stn;
        k_gemm_f32_small<Epi><<<stm * stn * P, 256, 0, s>>>(g);
        return true;
    } else {
        (void)g; (void)nb; (void)s;
        return false;
    }
}

template <typename T, int KA, int KB, class Epi, bool FAST, int NCH>
static void run_gemm(const morlax_ctx* c, int kind, GemmArgs<T, KA, KB, Epi, FAST, NCH>& g, int P, hipStream_t s) {
    if (g.crows == 0) g.crows = g.a.rows;
    if (g.ccols == 0) g.ccols = g.b.rows;
    g.tiles_m = (g.crows + BM - 1) / BM;
    g.tiles_n = (g.ccols + BN - 1) / BN;
    const int nb = g.tiles_m * g.tiles_n * P;
    GemmProf::Rec* r = prof_take(c, kind, 2.0 * g.crows * (double)g.ccols * g.a.kdim * (P / g.ranges));
    if (r) (void)hipEventRecord(r->a, s);
    if (!launch_special(g, P, nb, s)) k_grouped_gemm<T, KA, KB, Epi, FAST, NCH><<<nb, 256, 0, s>>>(g);
    if (r) (void)hipEventRecord(r->b, s);
}

// ---- output layer ------------------------------------------------------------------------------
// out = head(h W_L(p)^T + b_L(p)); actor: optional sampling a = mu + sigma eps and its log-density.
// A wave owns 16 rows; lane (row = lane % 16, chunk = lane / 16) feeds 16x16 MFMA tiles from global.
template <typename T>
__global__ __launch_bounds__(256) void k_head_fwd(const T* __restrict__ Hin, const T* __restrict__ theta_mat,
                                                 const float* __restrict__ theta_vec, int64_t mat_len,
                                                 int64_t vec_len, int64_t mat_off, int64_t vec_off, int W,
                                                 int out_dim, int M, int Mp, RowMap rm, int tanh_cols,
                                                 float* __restrict__ out, float* __restrict__ saved_out,
                                                 const float* __restrict__ eps, float* __restrict__ act,
                                                 float* __restrict__ logp, int64_t logsig_off, int adim,
                                                 int sig_state) {
    constexpr int VE = Elems<T>::VE;
    const int p = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = (blockIdx.x * 4 + wave) * 16;
    if (m0 >= M) return;
    const int lr = lane & 15, lg = lane >> 4;
    const T* hrow = Hin + ((int64_t)p * Mp + (m0 + lr)) * W;
    const T* wrow = theta_mat + (int64_t)p * mat_len + mat_off + (int64_t)lr * W;
    const bool a_ok = (m0 + lr) < M, b_ok = lr < out_dim;
    // eight contraction steps per batch: their loads are issued together, and two accumulators alternate so
    // that consecutive MFMAs do not wait for each other
    float4_t c = {0.f, 0.f, 0.f, 0.f}, c2 = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < W; k0 += 32 * VE) {
        uint4 fa[8], fb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + (4 * u + lg) * VE;
            fa[u] = make_uint4(0, 0, 0, 0);
            fb[u] = make_uint4(0, 0, 0, 0);
            if (a_ok && k < W) fa[u] = *reinterpret_cast<const uint4*>(hrow + k);
            if (b_ok && k < W) fb[u] = *reinterpret_cast<const uint4*>(wrow + k);
        }
#pragma unroll
        for (int u = 0; u < 8; u += 2) {
            Mma16<T>::run(fa[u], fb[u], c);
            Mma16<T>::run(fa[u + 1], fb[u + 1], c2);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] += c2[e];
    // lane holds column lr of rows m0 + 4*lg + e
    const float bias = b_ok ? theta_vec[(int64_t)p * vec_len + vec_off + lr] : 0.f;
    const bool mean_lane = lr < adim;  // lanes that hold an action mean
    float ls_p = 0.f;
    if (eps && mean_lane && !sig_state) ls_p = theta_vec[(int64_t)p * vec_len + logsig_off + lr];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int m = m0 + 4 * lg + e;
        const bool ok = (m < M) && b_ok;
        const float z = c[e] + bias;
        const float o = (lr < tanh_cols) ? tanhf(z) : z;
        int64_t row = 0;
        if (m < M) row = rm.row(p, m);
        float term = 0.f;
        // a state-dependent log sigma sits adim columns to the right, in the same group of 16 lanes
        const float ls_s = __shfl(o, (lane & 48) | ((lr + adim) & 15), 64);
        if (ok) {
            out[row * out_dim + lr] = o;
            if (saved_out) saved_out[((int64_t)p * M + m) * OUT_PITCH + lr] = o;
            if (eps && mean_lane) {
                const float ls = sig_state ? ls_s : ls_p;
                const float ep = eps[row * adim + lr];
                act[row * adim + lr] = o + expf(ls) * ep;
                term = -0.5f * ep * ep - ls;
            }
        }
        if (eps) {
            term += __shfl_xor(term, 8, 64);
            term += __shfl_xor(term, 4, 64);
            term += __shfl_xor(term, 2, 64);
            term += __shfl_xor(term, 1, 64);
            if (m < M && lr == 0) logp[row] = term - 0.918938533204672742f * (float)adim;
        }
    }
}

// ---- backward of the output layer, one launch -----------------------------------------------------------------
// dz_L = dout * (1 - mu^2) for the tanh head (else dout): four columns of row m of preference p, zero beyond out_dim
struct HeadDz {
    const float *dout, *saved_out;  // time-major [.., out_dim]; compact [P][M][OUT_PITCH]
    int32_t out_dim, tanh_cols, M;
    RowMap rm;
    struct Raw { float d[4], mu[4]; };
    __device__ inline void request(int p, int m, int q, Raw& r) const {
        const float* src = dout + rm.row(p, m) * out_dim;
        const float4 mu = *reinterpret_cast<const float4*>(saved_out + ((int64_t)p * M + m) * OUT_PITCH + 4 * q);
        r.mu[0] = mu.x; r.mu[1] = mu.y; r.mu[2] = mu.z; r.mu[3] = mu.w;
#pragma unroll
        for (int e = 0; e < 4; ++e) r.d[e] = src[4 * q + e < out_dim ? 4 * q + e : 0];
    }
    __device__ inline float value(const Raw& r, int q, int e, bool ok) const {
        const int j = 4 * q + e;
        float d = ok && j < out_dim ? r.d[e] : 0.f;
        if (j < tanh_cols) d *= (1.f - r.mu[e] * r.mu[e]);
        return ok ? d : 0.f;
    }
};

// Transposing 8-byte LDS read: the 16 lanes of a group address the 64-bit words of a 4 x 16 block of 16-bit values
// -- lane 4 e + c the word of contraction index e that holds columns 4 c .. 4 c + 3 -- and lane b of the group
// receives the four contraction indices of column b: the B operand of a 16x16x16 MFMA read from a row-major tile.
template <typename E>
__device__ inline short4_t lds_tr4(const E* word) {
    typedef __attribute__((address_space(3))) short4_t lds_s4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(word));
}

// Two roles, both bound by the streams they read (h; act'(z) and the stores of dZ):
//   dW  dW_L(p)[j, i] = sum_m dz_L[m, j] h_{L-1}[m, i]: a workgroup takes one of HB_SPLIT row ranges of one preference and
//       128 columns, and walks its rows 128 at a time: the dz rows (rounded to the GEMM input type) and the h tile sit in
//       LDS, the next ones are already on their way in registers; wave w multiplies dz^T [16 x 128] by h [128 x columns
//       32 w .. 32 w + 31]: bf16 networks with 16x16x16 bf16 MFMAs (dz^T staged with the contraction contiguous, h read
//       through transposing LDS reads), fp32 ones with 16x16x4 MFMAs.  Partials go to pw[p][range][j][i].
//   dZ  dZ_{L-1}[m, i] = (sum_j dz_L[m, j] W_L(p)[j, i]) * act'(z_{L-1})[m, i]: 64 rows x 128 columns a workgroup, 4 x 8 a
//       thread, with the column sums of the unrounded dZ over the 64 rows (the bias gradient of the layer below) and, the
//       first column's workgroups, of dz_L (that of the output layer).
// k_bwd_final adds the partials.  (As launches of their own behind one that wrote dz_L as compact rows: 20 + 78 + 109 us
// for 128 preferences x 2048 rows of width 512, here 185; 7.2 + 8.7 + 12.9 for 24 x 1250 of 256, here 17.4.)
#define HB_ROWS 128  // row ranges are whole multiples of this
#define HB_SPLIT 4
// rows of h (of dZ_0 in the narrow first layer's dW) that a workgroup stages at a time: with 128 fp32 rows its LDS and the
// next tile's registers leave a CU two workgroups, or one (16 preferences x 8192 rows x 256 in fp32, 64 rows instead of 128:
// 137 -> 128 us here, 59 -> 39 us in the first layer's dW; 10 x 1850 of 160: 23.6 -> 18.1 us here)
template <typename T> constexpr int hb_tile() { return sizeof(T) == 4 ? HB_ROWS / 2 : HB_ROWS; }
template <typename T>
struct HeadBwdLds {
    static constexpr int R = hb_tile<T>();
    static constexpr int HP = 128 + Elems<T>::VE;          // h tile pitch in elements (16 bytes of padding)
    static constexpr bool kBf = std::is_same<T, bf16_t>::value;
    float sdr[kBf ? 1 : R][MORLAX_MAX_OUT];                // fp32: dz rows as they lie
    bf16_t sdT[kBf ? MORLAX_MAX_OUT : 1][R + 8];           // bf16: dz^T, contraction contiguous
    T sh[R][HP];
};
struct HeadBwdLdsDz {
    float sdz[64][MORLAX_MAX_OUT], sdu[64][MORLAX_MAX_OUT + 1], red[16][128], sw[MORLAX_MAX_OUT][128];
};
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 4 : 2) void k_head_bwd(HeadDz hz, const T* __restrict__ Hin, const T* __restrict__ theta_mat,
                                                 int64_t mat_len, int64_t mat_off,
                                                 const typename GradT<T>::type* __restrict__ G, T* __restrict__ dZ,
                                                 float* __restrict__ pw, float* __restrict__ pb, float* __restrict__ part,
                                                 int W, int Mp, int n_front, int per_rest, RowDiv by_dw, RowDiv by_rest) {
    constexpr size_t kLds = sizeof(HeadBwdLds<T>) > sizeof(HeadBwdLdsDz) ? sizeof(HeadBwdLds<T>) : sizeof(HeadBwdLdsDz);
    __shared__ __align__(16) unsigned char lds[kLds];
    constexpr int VE = Elems<T>::VE;
    asm volatile("" ::"s"(hz.dout), "s"(theta_mat), "s"(n_front));  // (a value of each line of the arguments, as in k_bwd_final)
    const int ncol = (W + 127) / 128, M = hz.M;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // n_front dW workgroups ahead of everything else, or (0) every preference's ahead of its dZ ones (rule: the launch)
    const bool front = (int)blockIdx.x < n_front;
    const int id = front ? blockIdx.x : blockIdx.x - n_front;
    const int p = (int)(front ? by_dw : by_rest).quotient((uint32_t)id);
    int item = id - p * (front ? ncol * HB_SPLIT : per_rest);
    const bool dw_role = front || (n_front == 0 && item < ncol * HB_SPLIT);
    if (!dw_role && n_front == 0) item -= ncol * HB_SPLIT;
    const int i0 = item % ncol * 128;
    if (!dw_role) {
        HeadBwdLdsDz& L = *reinterpret_cast<HeadBwdLdsDz*>(lds);
        const int mb = item / ncol, m0 = mb * 64, n_mb = (Mp + 63) / 64;
        const int tr = (threadIdx.x / 16) * 4, ti = i0 + (threadIdx.x % 16) * 8;
        const bool live = ti < W;
        Pack8 gq[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int m = m0 + tr + a < Mp ? m0 + tr + a : Mp - 1;
            const uint4* src = reinterpret_cast<const uint4*>(G + ((int64_t)p * Mp + m) * W + (live ? ti : 0));
            gq[a].lo = src[0];
            if (sizeof(T) == 4) gq[a].hi = src[1];
        }
        // (W_L through LDS: read where it was needed it was a round trip to memory for every output, one behind the other; us a
        // backward pass of one hidden layer, so and here: 32 preferences x 8192 rows of 256 122 and 118, 24 x 1250 25.5 and 24.8)
        const int mm = threadIdx.x / 4, q = threadIdx.x % 4, m = m0 + mm;
        HeadDz::Raw raw;
        hz.request(p, m < M ? m : M - 1, q, raw);
        const int wj = threadIdx.x / 16;  // the thread's row of W_L, columns ti .. ti + 7
        Pack8 wq;
        {
            const uint4* src = reinterpret_cast<const uint4*>(theta_mat + (int64_t)p * mat_len + mat_off + (int64_t)(wj < hz.out_dim ? wj : 0) * W + (live ? ti : 0));
            wq.lo = src[0];
            if (sizeof(T) == 4) wq.hi = src[1];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d = hz.value(raw, q, e, m < M);
            L.sdu[mm][4 * q + e] = d;
            L.sdz[mm][4 * q + e] = to_f(cvt<T>(d));  // GEMM input rounding
        }
        {
            float wv[8];
            const uint32_t w[8] = {wq.lo.x, wq.lo.y, wq.lo.z, wq.lo.w, wq.hi.x, wq.hi.y, wq.hi.z, wq.hi.w};
#pragma unroll
            for (int b = 0; b < 8; ++b)
                wv[b] = __uint_as_float(sizeof(T) == 4 ? w[b] : (b & 1) ? w[b >> 1] & 0xffff0000u : w[b >> 1] << 16);
            store8(&L.sw[wj][threadIdx.x % 16 * 8], wv);
        }
        __syncthreads();
        float acc[4][8];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[a][b] = 0.f;
        for (int j = 0; j < hz.out_dim; ++j) {
            float wv[8];
            get8(&L.sw[j][threadIdx.x % 16 * 8], wv);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float d = L.sdz[tr + a][j];
#pragma unroll
                for (int b = 0; b < 8; ++b) acc[a][b] += d * wv[b];
            }
        }
        float cs[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) cs[b] = 0.f;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int m = m0 + tr + a;
            if (m >= Mp || !live) continue;  // (rows M .. Mp: their dz is zero, and so is dZ)
            float v[8], g[8];
            if constexpr (sizeof(T) == 2) {
                unpack8(gq[a].lo, g);
            } else {
                const uint32_t w[8] = {gq[a].lo.x, gq[a].lo.y, gq[a].lo.z, gq[a].lo.w, gq[a].hi.x, gq[a].hi.y, gq[a].hi.z, gq[a].hi.w};
#pragma unroll
                for (int b = 0; b < 8; ++b) g[b] = __uint_as_float(w[b]);
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                v[b] = acc[a][b] * g[b];
                cs[b] += v[b];
            }
            store8(dZ + ((int64_t)p * Mp + m) * W + ti, v);
        }
        // partial column sums of the unrounded dZ over this block's 64 rows (row groups in fixed order)
#pragma unroll
        for (int b = 0; b < 8; ++b) L.red[threadIdx.x / 16][(threadIdx.x % 16) * 8 + b] = cs[b];
        __syncthreads();
        if (threadIdx.x < 128 && i0 + threadIdx.x < W) {
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) v += L.red[q][threadIdx.x];
            part[((int64_t)p * n_mb + mb) * W + i0 + threadIdx.x] = v;
        }
        if (i0 == 0) {  // sums of dz_L over the 64 rows: a wave's butterfly, columns wave, wave + 4, ..
#pragma unroll
            for (int k = 0; k < MORLAX_MAX_OUT / 4; ++k) {
                float v = L.sdu[lane][wave + 4 * k];
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
                if (lane == 0) pb[((int64_t)p * n_mb + mb) * MORLAX_MAX_OUT + wave + 4 * k] = v;
            }
        }
        return;
    }
    HeadBwdLds<T>& L = *reinterpret_cast<HeadBwdLds<T>*>(lds);
    constexpr int CPR = 128 / VE;                          // 16-byte pieces per tile row
    constexpr int R = hb_tile<T>();                        // rows of a tile
    constexpr int NPT = R * CPR / 256;                     // pieces per thread
    constexpr int ND = R * 4 / 256;                        // quarter rows of dz per thread
    constexpr bool kBf = HeadBwdLds<T>::kBf;
    const int rs = item / ncol;
    const int per = ((M + HB_SPLIT - 1) / HB_SPLIT + HB_ROWS - 1) / HB_ROWS * HB_ROWS;  // rows per range
    const int m_lo = rs * per, m_hi = (m_lo + per < M) ? (m_lo + per) : M;
    const int ln = lane & 15, kg = lane >> 4;
    float4_t acc[2][2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[c][q] = float4_t{0.f, 0.f, 0.f, 0.f};
    uint4 nxt[NPT];
    HeadDz::Raw dnx[ND];
    auto fetch = [&](int m0) {
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int idx = threadIdx.x + 256 * i, m = m0 + idx / 4;
            hz.request(p, m < m_hi ? m : m_hi - 1, idx % 4, dnx[i]);
        }
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const int idx = threadIdx.x + 256 * q, mm = idx / CPR, cc = (idx % CPR) * VE;
            uint4 u = make_uint4(0, 0, 0, 0);
            if (m0 + mm < m_hi && i0 + cc < W)
                u = *reinterpret_cast<const uint4*>(Hin + ((int64_t)p * Mp + m0 + mm) * W + i0 + cc);
            nxt[q] = u;
        }
    };
    if (m_lo < m_hi) fetch(m_lo);
    for (int m0 = m_lo; m0 < m_hi; m0 += R) {
        __syncthreads();  // the previous tile has been multiplied
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int idx = threadIdx.x + 256 * i, mm = idx / 4, q = idx % 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const T d = cvt<T>(hz.value(dnx[i], q, e, m0 + mm < m_hi));
                if constexpr (kBf) L.sdT[4 * q + e][mm] = d;
                else L.sdr[mm][4 * q + e] = to_f(d);
            }
        }
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const int idx = threadIdx.x + 256 * q;
            *reinterpret_cast<uint4*>(&L.sh[idx / CPR][(idx % CPR) * VE]) = nxt[q];
        }
        if (m0 + R < m_hi) fetch(m0 + R);
        __syncthreads();
        if constexpr (kBf) {
            // both operands are bf16 values: 16x16x16 bf16 MFMAs, eight times the fp32 rate for the same sums
#pragma unroll
            for (int ks = 0; ks < R / 16; ++ks) {
                const short4_t a = *reinterpret_cast<const short4_t*>(&L.sdT[ln][16 * ks + 4 * kg]);  // dz^T[j = ln][4 m]
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[c][ks & 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                        a, lds_tr4(&L.sh[16 * ks + 4 * kg + (ln >> 2)][32 * wave + 16 * c + 4 * (ln & 3)]), acc[c][ks & 1], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < R / 4; ++kk) {
                const int m = 4 * kk + kg;
                const float a = L.sdr[m][ln];                              // dz^T[j = ln][m]
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float b = to_f(L.sh[m][32 * wave + 16 * c + ln]);  // h[m][column]
                    acc[c][kk & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[c][kk & 1], 0, 0, 0);
                }
            }
        }
    }
    // lane holds column ln of rows j = 4 kg + e
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int col = i0 + 32 * wave + 16 * c + ln;
        if (col < W) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                pw[(((int64_t)p * HB_SPLIT + rs) * MORLAX_MAX_OUT + 4 * kg + e) * W + col] = acc[c][0][e] + acc[c][1][e];
        }
    }
}

// ---- dW of a W x W layer with few preferences: contraction split into ranges ---------------------------------
// dW_l(p) has (W/128)^2 tiles per preference (the first layer fewer still) and the whole selection as its contraction;
// with few preferences that is a few dozen workgroups walking thousands of rows each.  The selection is cut into ranges
// that run as groups of the same grouped GEMM into partial matrices, and k_bwd_final adds the ranges in order.
#ifndef DW_SPLIT_TARGET
#define DW_SPLIT_TARGET 512
#endif
// ---- forward of the first layer with a narrow observation (O <= 32) ---------------------------------------
// h = act(x W0(p)^T + b0(p)) is, per output, an inner product of O terms: too short to fill GEMM tiles (the tiled
// kernel pads the contraction to 32 and loads the odd-width rows element by element) and bound by the stores of h
// and act'(z).  A block of 256 threads takes FN_ROWS rows of one preference with W0(p) in LDS, transposed to
// [i][o] in fp32 (exact for bf16 weights), and the rows' observations rounded to the network's type as the GEMM
// rounds them; a thread owns eight consecutive outputs of FN_ROWS / RPT rows, walks the contraction once with its
// eight weights of the step in registers, and stores 16- or 32-byte pieces that the threads of a row join to whole
// rows.  Sums run in ascending i in fp32, as one accumulator per output.
#define FN_ROWS 64
template <typename T, int ACT, bool SAVE>
__global__ __launch_bounds__(256) void k_first_fwd_narrow(const float* __restrict__ x, const T* __restrict__ theta_mat,
                                                         const float* __restrict__ theta_vec, int64_t mat_len,
                                                         int64_t vec_len, int64_t mat_off, int64_t vec_off, int O, int W,
                                                         int M, int Mp, RowMap rm, T* __restrict__ H,
                                                         typename GradT<T>::type* __restrict__ G) {
    extern __shared__ __align__(16) float fn_lds[];
    const int WP = W + 4;  // pitch of a row of W0^T: keeps 16-byte alignment, shifts the banks from row to row
    float* sw = fn_lds;               // [O][WP]
    float* sb = sw + O * WP;          // [W]
    float* sx = sb + W;               // [FN_ROWS][O]
    const int p = blockIdx.y, m0 = blockIdx.x * FN_ROWS;
    const T* w0 = theta_mat + (int64_t)p * mat_len + mat_off;
    for (int idx = threadIdx.x; idx < W * O; idx += 256) {
        const int o = idx / O, i = idx - o * O;
        sw[i * WP + o] = to_f(w0[idx]);
    }
    for (int o = threadIdx.x; o < W; o += 256) sb[o] = theta_vec[(int64_t)p * vec_len + vec_off + o];
    for (int idx = threadIdx.x; idx < FN_ROWS * O; idx += 256) {
        const int r = idx / O, i = idx - r * O;
        const int m = m0 + r < M ? m0 + r : M - 1;
        sx[idx] = to_f(cvt<T>(x[rm.row(p, m) * O + i]));
    }
    __syncthreads();
    const int CH = W >> 3;        // pieces of eight outputs per row (at most 256)
    const int RPT = 256 / CH;     // rows in work at a time
    const int chunk = threadIdx.x % CH, slot = threadIdx.x / CH;
    if (slot >= RPT) return;
    constexpr int TURNS = 8;      // rows per thread and pass
    for (int r0 = 0; r0 < FN_ROWS; r0 += RPT * TURNS) {
        float acc[TURNS][8];
        const float4 b0 = *reinterpret_cast<const float4*>(sb + 8 * chunk), b1 = *reinterpret_cast<const float4*>(sb + 8 * chunk + 4);
        const float* xr[TURNS];
#pragma unroll
        for (int t = 0; t < TURNS; ++t) {
            acc[t][0] = b0.x; acc[t][1] = b0.y; acc[t][2] = b0.z; acc[t][3] = b0.w;
            acc[t][4] = b1.x; acc[t][5] = b1.y; acc[t][6] = b1.z; acc[t][7] = b1.w;
            const int r = r0 + slot + t * RPT;
            xr[t] = sx + (r < FN_ROWS ? r : FN_ROWS - 1) * O;
        }
        for (int i = 0; i < O; ++i) {  // (the observation values read four steps at a time measured no faster)
            const float4 wa = *reinterpret_cast<const float4*>(sw + i * WP + 8 * chunk);
            const float4 wb = *reinterpret_cast<const float4*>(sw + i * WP + 8 * chunk + 4);
#pragma unroll
            for (int t = 0; t < TURNS; ++t) {
                const float xv = xr[t][i];
                acc[t][0] += xv * wa.x; acc[t][1] += xv * wa.y; acc[t][2] += xv * wa.z; acc[t][3] += xv * wa.w;
                acc[t][4] += xv * wb.x; acc[t][5] += xv * wb.y; acc[t][6] += xv * wb.z; acc[t][7] += xv * wb.w;
            }
        }
#pragma unroll
        for (int t = 0; t < TURNS; ++t) {
            const int r = r0 + slot + t * RPT, m = m0 + r;
            if (r < FN_ROWS && m < Mp) {
                float g[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) act_pair<T, ACT, true>(acc[t][u], acc[t][u], g[u]);
                const int64_t at = ((int64_t)p * Mp + m) * W + 8 * chunk;
                put8(H + at, pack8(acc[t], (const T*)nullptr));
                if (SAVE) put8(G + at, pack8(g, (const typename GradT<T>::type*)nullptr));
            }
        }
    }
}
static int64_t first_fwd_narrow_lds(const morlax_ctx* c) {
    return ((int64_t)(c->d.width + 4) * c->d.obs_dim + c->d.width + (int64_t)FN_ROWS * c->d.obs_dim) * 4;
}
static bool first_fwd_narrow_ok(const morlax_ctx* c) {
    // bf16 networks only: with fp32 outputs (twice the bytes per store) the tiled kernel measured faster
    return c->d.wdtype == 1 && c->d.obs_dim <= 32 && c->d.width % 8 == 0 && c->d.width <= 2048 &&
           first_fwd_narrow_lds(c) <= 64 * 1024;
}

// ---- first layer with a narrow observation (O <= 32) and few preferences ----------------------------------
// dW_0(p)[o, i] = sum_m dZ_0[m, o] x[m, i] has W x O outputs and the whole selection as its contraction: as a tiled
// GEMM it is two or three tiles per preference walking thousands of rows each (workload 2: 32 workgroups on 256 CUs).
// It is the output layer's dW with the roles exchanged, so it takes the same streaming form: a block takes one of n_split
// row ranges of one preference and 128 columns of dZ_0, gathers the observation rows through the row map (the offsets of
// the next tile's rows in LDS, the rows' values one after the other: consecutive threads read consecutive floats of an
// environment's run) into 16 JB columns, zero beyond O, and k_bwd_final adds the ranges in order.  (The rows gathered by a
// launch of their own first: 14.2 + 29.2 us for 32 preferences x 8192 rows x 11 x 256, here 31.1.)
template <typename T, int JB>
__global__ __launch_bounds__(256) void k_first_bwd_dw(const float* __restrict__ x, const T* __restrict__ dZ,
                                                     float* __restrict__ pw, int O, int W, int M, int Mp, int n_split,
                                                     RowMap rm) {
    constexpr int VE = Elems<T>::VE;
    constexpr int HP = 128 + VE;
    constexpr int CPR = 128 / VE;
    constexpr int R = hb_tile<T>();         // rows of a tile
    constexpr int NPT = R * CPR / 256;
    constexpr int OP = 16 * JB;
    constexpr int NX = R * OP / 256;  // observation values per thread, at most
    constexpr bool kBf = std::is_same<T, bf16_t>::value;
    __shared__ __align__(16) float sdr[kBf ? 1 : R][OP];        // fp32: observation rows as they lie
    __shared__ __align__(16) bf16_t sdT[kBf ? OP : 1][R + 8];  // bf16: x^T, contraction contiguous
    __shared__ __align__(16) T sh[R][HP];
    __shared__ uint32_t sro[2][R];  // first element of a tile row's observation
    const int p = blockIdx.z, rs = blockIdx.y, i0 = blockIdx.x * 128;
    const int per = ((M + n_split - 1) / n_split + HB_ROWS - 1) / HB_ROWS * HB_ROWS;  // rows per range
    const int m_lo = rs * per, m_hi = (m_lo + per < M) ? (m_lo + per) : M;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, kg = lane >> 4;
    float4_t acc[JB][2][2];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[jb][c][q] = float4_t{0.f, 0.f, 0.f, 0.f};
    uint4 nxt[NPT];
    float xn[NX];
    const int mm0 = threadIdx.x / O, c0 = threadIdx.x % O, dm = 256 / O, dc = 256 % O;  // value i + 1 of a thread: 256 further
    auto each_x = [&](auto fn) {
        int mm = mm0, c = c0;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            if (mm < R) fn(i, mm, c);
            mm += dm; c += dc;
            if (c >= O) { c -= O; ++mm; }
        }
    };
    auto offsets = [&](int m0, int slot) {
        if (threadIdx.x < R) {
            const int m = m0 + (int)threadIdx.x;
            sro[slot][threadIdx.x] = (uint32_t)(rm.row(p, m < m_hi ? m : m_hi - 1) * O);
        }
    };
    auto fetch = [&](int m0, int slot) {
        each_x([&](int i, int mm, int c) { xn[i] = x[sro[slot][mm] + c]; });
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const int idx = threadIdx.x + 256 * q, mm = idx / CPR, cc = (idx % CPR) * VE;
            uint4 u = make_uint4(0, 0, 0, 0);
            if (m0 + mm < m_hi && i0 + cc < W)
                u = *reinterpret_cast<const uint4*>(dZ + ((int64_t)p * Mp + m0 + mm) * W + i0 + cc);
            nxt[q] = u;
        }
    };
    for (int idx = threadIdx.x; idx < R * (OP - O); idx += 256) {  // columns beyond O
        const int mm = idx % R, c = O + idx / R;
        if constexpr (kBf) sdT[c][mm] = (bf16_t)0.f;
        else sdr[mm][c] = 0.f;
    }
    if (m_lo < m_hi) {
        offsets(m_lo, 0);
        __syncthreads();
        fetch(m_lo, 0);
    }
    for (int m0 = m_lo, slot = 0; m0 < m_hi; m0 += R, slot ^= 1) {
        __syncthreads();  // the previous tile has been multiplied
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const int idx = threadIdx.x + 256 * q;
            *reinterpret_cast<uint4*>(&sh[idx / CPR][(idx % CPR) * VE]) = nxt[q];
        }
        each_x([&](int i, int mm, int c) {
            const T v = cvt<T>(m0 + mm < m_hi ? xn[i] : 0.f);  // GEMM input rounding
            if constexpr (kBf) sdT[c][mm] = v;
            else sdr[mm][c] = to_f(v);
        });
        if (m0 + R < m_hi) offsets(m0 + R, slot ^ 1);
        __syncthreads();
        if (m0 + R < m_hi) fetch(m0 + R, slot ^ 1);
        if constexpr (kBf) {
#pragma unroll
            for (int ks = 0; ks < R / 16; ++ks) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const short4_t b = lds_tr4(&sh[16 * ks + 4 * kg + (ln >> 2)][32 * wave + 16 * c + 4 * (ln & 3)]);
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        acc[jb][c][ks & 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                            *reinterpret_cast<const short4_t*>(&sdT[16 * jb + ln][16 * ks + 4 * kg]), b, acc[jb][c][ks & 1], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < R / 4; ++kk) {
                const int m = 4 * kk + kg;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float b = to_f(sh[m][32 * wave + 16 * c + ln]);  // dZ_0[m][column]
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        acc[jb][c][kk & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(sdr[m][16 * jb + ln], b, acc[jb][c][kk & 1], 0, 0, 0);
                }
            }
        }
    }
    // lane holds column ln of observation components 16 jb + 4 kg + e
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int col = i0 + 32 * wave + 16 * c + ln;
            if (col < W) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    pw[(((int64_t)p * n_split + rs) * OP + 16 * jb + 4 * kg + e) * W + col] = acc[jb][c][0][e] + acc[jb][c][1][e];
            }
        }
}

// What the backward launches of a network leave as partial sums, added up by one launch at their end (one behind each of
// them put some fifteen launches of 4 - 10 us on the dependent chain of a network's gradients).  Blocks of a preference, in
// this order:
//   bias sums  db_l(p)[o]: 32 columns of one layer; its eight groups of 32 threads each add a contiguous eighth of the row
//              blocks in order, and the eight sums are added in group order
//   output layer's dW (ranges in order); its first block also the bias sums (64-row sums, four to a block of 256 rows, the
//              blocks in order) and the copy of the log-sigma gradient
//   split dW   the ranges of a layer whose contraction was split, in order, four elements a thread
//   first dW   the ranges' partials [i][o] of the narrow first layer, in order
// Fixed associations throughout: results repeat bit for bit.
// Bound by latency where the partials are few and by memory where they are many, so a thread requests up to 32 terms of its sum
// together, those behind the last one the last one once more, and the narrow first layer's partials are read along their rows and
// turned in LDS; where they are few the reads of its arguments, some ten lines of host memory, are the larger part, and are on their
// way together too.  us a launch, in loops of two to four requests, and so: 16 preferences x 8192 rows of 3 x 256, fp32, 8 ranges 32.8 and
// 20.4; 32 of them, bf16, 4 ranges 26.2 and 22.2; 64 x 4096 of 4 x 512 16.1 and 15.0; 24 x 1250 of 3 x 256 4.1 and 3.7; 4 x 256 of 2 x 32
// 3.7 and 3.0; 112 x 84 of 4 x 160 4.2 and 5.2.
struct BwdFinalArgs {
    const float *part, *dlogsig;
    float *dmat, *dvec;
    int64_t mat_len, vec_len;
    int32_t W, L, O, OP, out_dim, A;  // A: log-sigma components to write, 0: none
    int32_t n_part[MORLAX_MAX_LAYERS], S[MORLAX_MAX_LAYERS], n_pb, first_ns;  // S: ranges of a split dW, 1: not split
    int64_t colsum[MORLAX_MAX_LAYERS], split[MORLAX_MAX_LAYERS], first, pw, pb;  // offsets in part
    int64_t mat_off[MORLAX_MAX_LAYERS], vec_off[MORLAX_MAX_LAYERS], n[MORLAX_MAX_LAYERS], logsig_off;  // (index L: output layer)
    int32_t b_head, b_split[MORLAX_MAX_LAYERS], b_first;  // first block of each kind
};
// N of the terms at(0) .. at(n - 1) from q on, requested together
template <int N, typename V, typename At>
__device__ inline void get_terms(V (&v)[N], int q, int n, const At& at) {
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = at(q + u < n ? q + u : n - 1);
}
// add(at(lo)), .. add(at(hi - 1)) in order, so many requested together as there are: FEW or MANY
template <int N, typename V, typename At, typename Add>
__device__ inline void each_term(int lo, int hi, const At& at, const Add& add) {
    for (int q = lo; q < hi; q += N) {
        V v[N];
        get_terms(v, q, hi, at);
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (q + u < hi) add(v[u]);
    }
}
template <int FEW, int MANY, typename V, typename At, typename Add>
__device__ inline void in_order(int lo, int hi, int n, const At& at, const Add& add) {
    if (n <= FEW) each_term<FEW, V>(lo, hi, at, add);
    else each_term<MANY, V>(lo, hi, at, add);
}
__global__ __launch_bounds__(256) void k_bwd_final(BwdFinalArgs a) {
    __shared__ float sg[8][33];
    // a value of each 64-byte line of the arguments (host memory, half a microsecond the first time a workgroup reads a line), all on
    // their way together
    asm volatile("" ::"s"(a.W), "s"(a.n_part[0]), "s"(a.n_pb), "s"((int)a.colsum[MORLAX_MAX_LAYERS - 1]), "s"((int)a.first),
                 "s"((int)a.mat_off[0]), "s"((int)a.vec_off[0]), "s"((int)a.n[0]), "s"(a.b_head), "s"(a.b_first));
    const int p = blockIdx.y, b = blockIdx.x, W = a.W;
    float* dmat = a.dmat + (int64_t)p * a.mat_len;
    float* dvec = a.dvec + (int64_t)p * a.vec_len;
    if (b < a.b_head) {
        const int cw = (W + 31) / 32, l = b / cw, np = a.n_part[l];
        const int c = threadIdx.x & 31, g = threadIdx.x >> 5, i = (b - l * cw) * 32 + c;
        const float* part = a.part + a.colsum[l] + (int64_t)p * np * W + (i < W ? i : W - 1);
        const int per = (np + 7) / 8, q_lo = g * per, q_hi = (q_lo + per < np) ? q_lo + per : np;
        float t = 0.f;
        auto at = [&](int q) { return part[(int64_t)q * W]; };
        auto add = [&](float v) { t += v; };
        if (per == 1) each_term<1, float>(q_lo, q_hi, at, add);
        else in_order<4, 8, float>(q_lo, q_hi, per, at, add);
        sg[g][c] = t;
        __syncthreads();
        if (g == 0 && i < W) {
            t = sg[0][c];
#pragma unroll
            for (int k = 1; k < 8; ++k) t += sg[k][c];
            dvec[a.vec_off[l] + i] = t;
        }
        return;
    }
    if (b < a.b_split[0]) {
        const int idx = (b - a.b_head) * 256 + threadIdx.x;
        if (idx < a.out_dim * W) {
            const int j = idx / W, i = idx % W;
            float v = 0.f;
#pragma unroll
            for (int c = 0; c < HB_SPLIT; ++c) v += a.part[a.pw + (((int64_t)p * HB_SPLIT + c) * MORLAX_MAX_OUT + j) * W + i];
            dmat[a.mat_off[a.L] + idx] = v;
        }
        if (idx < a.out_dim) {
            const float* pb = a.part + a.pb + (int64_t)p * a.n_pb * MORLAX_MAX_OUT + idx;
            float v = 0.f;
            auto add = [&](auto some) __attribute__((always_inline)) {
                constexpr int N = decltype(some)::value;  // sums of 64 rows requested together
                for (int m = 0; m < a.n_pb; m += N) {
                    float t[N];
                    get_terms(t, m, a.n_pb, [&](int q) { return pb[(int64_t)q * MORLAX_MAX_OUT]; });
                    auto at = [&](int u) { return m + u < a.n_pb ? t[u] : 0.f; };
#pragma unroll
                    for (int u = 0; u < N; u += 4)
                        if (m + u < a.n_pb) v += (at(u) + at(u + 1)) + (at(u + 2) + at(u + 3));
                }
            };
            if (a.n_pb <= 4) add(std::integral_constant<int, 4>{});
            else add(std::integral_constant<int, 32>{});
            dvec[a.vec_off[a.L] + idx] = v;
        }
        if (idx < a.A) dvec[a.logsig_off + idx] = a.dlogsig ? a.dlogsig[p * a.A + idx] : 0.f;
        return;
    }
    if (b < a.b_first) {
        int l = 0;
#pragma unroll
        for (int k = 1; k < MORLAX_MAX_LAYERS; ++k) l = k < a.L && b >= a.b_split[k] ? k : l;
        const int64_t n = a.n[l], i4 = ((int64_t)(b - a.b_split[l]) * 256 + threadIdx.x) * 4;
        if (i4 >= n) return;
        const int S = a.S[l];
        const float* src = a.part + a.split[l] + (int64_t)p * S * n + i4;
        float v[4];
        auto at = [&](int c) { return *reinterpret_cast<const u32x4_t*>(src + c * n); };
        auto add = [&](const u32x4_t& u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += __uint_as_float(u[e]);
        };
        const u32x4_t first = at(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(first[e]);
        in_order<3, 7, u32x4_t>(1, S, S - 1, at, add);
        // W is a multiple of 16, so every matrix starts on a 16-byte boundary of the row
        *reinterpret_cast<float4*>(dmat + a.mat_off[l] + i4) = make_float4(v[0], v[1], v[2], v[3]);
        return;
    }
    // eight inputs x 32 features, read along the partials' rows and turned in LDS: every access is a run of 32 bytes or more
    const int cw = (W + 31) / 32, it = (b - a.b_first) / cw, o0 = (b - a.b_first - it * cw) * 32, i0 = it * 8;
    {
        const int c = threadIdx.x & 31, g = threadIdx.x >> 5, o = o0 + c < W ? o0 + c : W - 1, i = i0 + g < a.O ? i0 + g : a.O - 1;
        const float* src = a.part + a.first + ((int64_t)p * a.first_ns * a.OP + i) * W + o;
        float v = 0.f;
        in_order<4, 16, float>(0, a.first_ns, a.first_ns, [&](int q) { return src[(int64_t)q * a.OP * W]; }, [&](float t) { v += t; });
        sg[g][c] = v;
    }
    __syncthreads();
    const int o = o0 + (threadIdx.x >> 3), i = i0 + (threadIdx.x & 7);
    if (o < W && i < a.O) dmat[a.mat_off[0] + (int64_t)o * a.O + i] = sg[threadIdx.x & 7][threadIdx.x >> 3];
}

// Rows of the fp32 observation tensor picked by the row map, rounded to the GEMM input type, as compact
// [P][Mp][ldx] rows (ldx a multiple of 8): zeros beyond O, copies of row M - 1 beyond M.
template <typename T>
__global__ __launch_bounds__(256) void k_gather_x(const float* __restrict__ x, T* __restrict__ xc, int O, int ldx, int M,
                                                 int Mp, RowMap rm) {
    const int p = blockIdx.y;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // one 8-element piece
    const int per_row = ldx / 8;
    if (idx >= (int64_t)Mp * per_row) return;
    const int m = (int)(idx / per_row), c = (int)(idx % per_row) * 8;
    const float* src = x + rm.row(p, m < M ? m : M - 1) * O + c;
    float v[8];
    if ((O & 7) == 0) {
        get8(src, v);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c + e < O ? src[e] : 0.f;
    }
    store8(xc + ((int64_t)p * Mp + m) * ldx + c, v);
}

// ---- host side ---------------------------------------------------------------------------------
static int64_t esize(const morlax_ctx* c) { return c->d.wdtype == 1 ? 2 : 4; }
// Rows per preference of the compact buffers (h, act', dZ, observations): whole contraction steps of the dW products.
// Rows M .. Mp are zero in dZ and what h, act' and the observations hold there is finite where row M - 1 and the biases are
// (copies of row M - 1; behind the tiled first layer of an odd observation width, the activation of the bias alone), so
// they add nothing.  (With Mp = M, a selection that was no multiple of 32 rows took the register-staged GEMM with a masked
// tail: 41 us against 18 us per launch at 24 preferences x 1250 rows x 256 x 256 in bf16, both unsplit; where the first
// layer's operand was read through the row map element by element, 334 us.)
static int pad_rows(const RowSel& rs) { return (rs.M + 31) / 32 * 32; }
static int64_t act_elems(const morlax_ctx* c, const RowSel& rs) {
    return align_up((int64_t)c->d.P * pad_rows(rs) * c->d.width, 64);
}

static int x0_ld(const morlax_ctx* c) { return (c->d.obs_dim + 7) / 8 * 8; }
static int64_t x0_elems(const morlax_ctx* c, const RowSel& rs) {
    return align_up((int64_t)c->d.P * pad_rows(rs) * x0_ld(c), 64);
}
// layer-by-layer forward from the compact first-layer input: bf16 networks whose observation width suits the
// direct-to-LDS GEMMs
static bool use_x0(const morlax_ctx* c) { return c->d.wdtype == 1 && c->d.obs_dim % 32 == 0; }
// the first layer's dW as a streaming split-K kernel: narrow observations and too few GEMM tiles to fill the chip; any
// other first layer's dW is a grouped GEMM on the compact observations the forward pass saved
static bool first_skinny(const morlax_ctx* c) {
    return c->d.obs_dim <= 32 && ((c->d.width + 127) / 128) * c->d.P < 256;
}
// saved: per hidden layer h and act', then the head's output rows, then (when used) the gathered observations
static int64_t saved_x0_off(const morlax_ctx* c, const RowSel& rs) {
    return 2 * (int64_t)c->d.n_hidden * act_elems(c, rs) * esize(c) + align_up((int64_t)c->d.P * rs.M * OUT_PITCH * 4, 256);
}
int64_t mlp_saved_bytes(const morlax_ctx* c, int net, const RowSel& rs) {
    (void)net;
    return saved_x0_off(c, rs) + (first_skinny(c) ? 0 : x0_elems(c, rs) * esize(c));
}
static int first_split(const morlax_ctx* c, const RowSel& rs) {
    const int tiles = ((c->d.width + 127) / 128) * c->d.P;
    int n = (1024 + tiles - 1) / tiles;
    const int cap = (rs.M + HB_ROWS - 1) / HB_ROWS;
    n = n > 64 ? 64 : n;
    n = n > cap ? cap : n;
    return n < 1 ? 1 : n;
}
// Ranges the contraction of a layer's dW is cut into (1 = the plain grouped GEMM), until there are DW_SPLIT_TARGET
// workgroups (1024 measured slower: twice the partials).  fp32: ranges of 256 rows and more, of 64 while the workgroups
// reach less than a quarter of the CUs (4 preferences x 256 rows x 64 x 64: 10.9 us unsplit, 6.8
// split; the backward pass, the ranges added by k_bwd_final, 34.0 and 29.7).
// bf16: hidden layers only into equal ranges of whole 64-row steps, 256 rows and more; the first layer, whose few columns
// make few tiles, into ranges of 2048 rows and more, uneven ones too.  Uneven ranges of a bf16 hidden layer were timed at
// one shape only, which has more tiles than the chip has CUs (23 preferences x 1120 rows x 512 x 512 in two: 4 % of the
// update step lost); where few tiles leave the chip idle nothing was measured, and such a selection runs unsplit.  The room
// for the partials is sized for the most ranges any smaller selection takes.
static int dw_split(const morlax_ctx* c, int M, int layer, bool room) {
    const bool bf = c->d.wdtype == 1;
    const int d_in = layer == 0 ? c->d.obs_dim : c->d.width;
    const int64_t tiles = (int64_t)((c->d.width + 127) / 128) * ((d_in + 127) / 128) * c->d.P;
    int S = 1;
    while (S < 16 && tiles * S < DW_SPLIT_TARGET) {
        const int rows = bf ? (layer == 0 ? 2048 : 256) : (tiles * S < 64 ? 64 : 256);
        if (M / (2 * S) < rows || (bf && layer > 0 && !room && M % (2 * S * 64))) break;
        S *= 2;
    }
    return S;
}
static int dw_range(const RowSel& rs, int S) { return (int)align_up((pad_rows(rs) + S - 1) / S, 64); }
// fp32 scratch behind the two activation buffers: the partial sums of a network's backward launches, each in a place of
// its own until k_bwd_final has added it up (offsets in floats)
struct BwdPart {
    int64_t pw, pb, first, total;
    int64_t colsum[MORLAX_MAX_LAYERS], split[MORLAX_MAX_LAYERS];
};
static BwdPart bwd_part(const morlax_ctx* c, const RowSel& rs) {
    const int64_t P = c->d.P, W = c->d.width, n64 = (pad_rows(rs) + 63) / 64;
    BwdPart B;
    int64_t at = 0;
    auto take = [&](int64_t n) { const int64_t o = at; at += align_up(n, 64); return o; };
    B.pw = take(P * HB_SPLIT * MORLAX_MAX_OUT * W);
    B.pb = take(P * n64 * MORLAX_MAX_OUT);
    B.first = take(first_skinny(c) ? P * first_split(c, rs) * (c->d.obs_dim <= 16 ? 16 : 32) * W : 0);
    for (int l = 0; l < c->d.n_hidden; ++l) {
        const int S = dw_split(c, rs.M, l, true);
        B.colsum[l] = take(P * n64 * W);
        B.split[l] = take(S > 1 ? P * S * W * (l == 0 ? c->d.obs_dim : W) : 0);
    }
    B.total = at;
    return B;
}
static int64_t part_elems(const morlax_ctx* c, const RowSel& rs) { return bwd_part(c, rs).total; }
static bool fused_fwd_dims_ok(const morlax_ctx* c) {
    return c->d.wdtype == 1 && (c->d.width == 512 || c->d.width == 256) && c->d.obs_dim <= c->d.width &&
           c->d.n_hidden >= 1;
}
// elements per preference of the fused forward's copy of the matrices: the first layer's rows padded to a multiple of 64
static int64_t fused_frag_len(const morlax_ctx* c, int net) {
    const int Opad = (c->d.obs_dim + 63) & ~63;
    return c->net[net].mat_len + (int64_t)c->d.width * (Opad - c->d.obs_dim);
}

int64_t mlp_ws_bytes(const morlax_ctx* c, const RowSel& rs) {
    int64_t b = 2 * act_elems(c, rs) * esize(c) + part_elems(c, rs) * 4 + (use_x0(c) ? x0_elems(c, rs) * esize(c) : 0);
    if (fused_fwd_dims_ok(c)) {  // the fused forward's copy of the matrices in fragment order
        for (int net = 0; net < 2; ++net) {
            const int64_t f = align_up((int64_t)c->d.P * fused_frag_len(c, net) * 2, 256);
            if (f > b) b = f;
        }
    }
    return b;
}

static RowMap make_rowmap(const morlax_ctx* c, const RowSel& rs) {
    RowMap rm;
    rm.t0 = rs.t0; rm.j0 = rs.j0; rm.j_cnt = rs.j_cnt; rm.N = c->d.N; rm.n_g = c->n_g;
    rm.by = rs.by;
    return rm;
}

// The fused forward serves bf16 networks of width 512 or 256 (the observation is zero-filled to a multiple of 64 in LDS).
static bool fused_fwd_ok(const morlax_ctx* c, const NetDev& nd, const void* theta_mat) {
    if (!fused_fwd_dims_ok(c)) return false;
    if ((reinterpret_cast<uintptr_t>(theta_mat) & 15) || (nd.mat_len & 7)) return false;
    for (int l = 0; l <= c->d.n_hidden; ++l)
        if (nd.layer[l].mat_off & 7) return false;
    return true;
}

template <int ACT, bool SAVE, int WD>
static void launch_fused_fwd_w(const morlax_ctx* c, const FusedFwdArgs& a, hipStream_t s) {
    constexpr int lds = FF_ROWS * WD * 2 + (SAVE ? (WD / 64) * 4096 : 0);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_fused_fwd<ACT, SAVE, WD>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    const double per_row = 2.0 * WD * ((double)a.O + (double)(a.L - 1) * WD);
    GemmProf::Rec* r = prof_take(c, 5, per_row * a.M * c->d.P);
    if (r) (void)hipEventRecord(r->a, s);
    // width 512: one workgroup per CU (the tile fills its LDS); width 256: half the tile and half the waves, two per CU
    const int slots = resident_slots() / 2 * (512 / WD);
    k_mlp_fused_fwd<ACT, SAVE, WD><<<a.n_tiles < slots ? a.n_tiles : slots, WD, lds, s>>>(a);
    if (r) (void)hipEventRecord(r->b, s);
}
template <int ACT, bool SAVE>
static void launch_fused_fwd(const morlax_ctx* c, const FusedFwdArgs& a, hipStream_t s) {
    if (c->d.width == 256) launch_fused_fwd_w<ACT, SAVE, 256>(c, a, s);
    else launch_fused_fwd_w<ACT, SAVE, 512>(c, a, s);
}

static void fill_fwd_net(const morlax_ctx* c, int net, const void* theta_mat, const float* theta_vec, const RowSel& rs,
                         float* out, float* saved_out, const float* eps, float* act, float* logp, char* H, char* G,
                         char* x0, FwdNet& n) {
    const NetDev& nd = c->net[net];
    const LayerDev& Lo = nd.layer[c->d.n_hidden];
    n.theta_mat = theta_mat; n.theta_vec = theta_vec;
    n.mat_len = nd.mat_len; n.vec_len = nd.vec_len;
    n.head_mat_off = Lo.mat_off; n.head_vec_off = Lo.vec_off; n.logsig_off = Lo.vec_off + Lo.d_out;
    n.out_dim = nd.out_dim;
    n.tanh_cols = (net == MORLAX_ACTOR && c->d.mean_tanh) ? c->d.act_dim : 0;
    n.adim = c->d.act_dim;
    n.sig_state = (net == MORLAX_ACTOR && c->d.sigma_state) ? 1 : 0;
    n.M = rs.M; n.rm = make_rowmap(c, rs);
    n.out = out; n.saved_out = saved_out; n.eps = eps; n.act = act; n.logp = logp;
    n.H = H; n.G = G; n.x0 = x0;
}

static void run_mlp_fwd(const morlax_ctx* c, const NetDev& nd, FwdArgs& a, int rt, bool save, hipStream_t s) {
    const int W = c->d.width, L = c->d.n_hidden, O = c->d.obs_dim, P = c->d.P;
    a.L = L; a.O = O; a.W = W; a.act = c->d.act;
    a.perm = fused_fwd_ok(c, nd, a.net.theta_mat) ? 1 : 0;
    a.narrow = !a.perm && !use_x0(c) && first_fwd_narrow_ok(c) ? 1 : 0;
    const int th = a.split ? 32 * a.split : 16 * fwd_compiled((int)esize(c), fwd_waves(W), rt);
    a.net.tiles_m = ((save ? a.Mp : a.net.M) + th - 1) / th;
    const int n_tiles = a.net.tiles_m * P;
    GemmProf::Rec* r = prof_take(c, 5, 2.0 * W * ((double)O + (double)(L - 1) * W) * a.net.M * P);
    if (r) (void)hipEventRecord(r->a, s);
    if (c->d.wdtype == 1) {
        if (save) launch_mlp_fwd_bf16_save(a, rt, n_tiles, s);
        else launch_mlp_fwd_bf16_act(a, rt, n_tiles, s);
    } else {
        if (save) launch_mlp_fwd_f32_save(a, rt, n_tiles, s);
        else launch_mlp_fwd_f32_act(a, rt, n_tiles, s);
    }
    if (r) (void)hipEventRecord(r->b, s);
}

template <typename T>
static void policy_fwd_t(const morlax_ctx* c, int net, const T* theta_mat, const float* theta_vec, const float* x,
                         const RowSel& rs, float* out, const float* eps, float* act, float* logp, void* saved,
                         void* ws, hipStream_t s) {
    const NetDev& nd = c->net[net];
    const int P = c->d.P, W = c->d.width, M = rs.M, L = c->d.n_hidden, O = c->d.obs_dim;
    const int Mp = pad_rows(rs);
    const int64_t ae = act_elems(c, rs);
    const RowMap rm = make_rowmap(c, rs);
    T* sv = reinterpret_cast<T*>(saved);
    T* sv_x0 = (sv && !first_skinny(c)) ? reinterpret_cast<T*>(reinterpret_cast<char*>(sv) + saved_x0_off(c, rs)) : nullptr;
    T* wsT = reinterpret_cast<T*>(ws);
    auto Hbuf = [&](int l) { return sv ? sv + (int64_t)(2 * l) * ae : wsT + (int64_t)(l & 1) * ae; };
    typedef typename GradT<T>::type GT;
    auto Gbuf = [&](int l) { return sv ? reinterpret_cast<GT*>(sv + (int64_t)(2 * l + 1) * ae) : (GT*)nullptr; };
    float* saved_out = sv ? reinterpret_cast<float*>(sv + (int64_t)2 * L * ae) : nullptr;
    constexpr int VE = Elems<T>::VE;
    auto layer = [&](int l, auto act_tag, auto save_tag) {
        constexpr int ACT = decltype(act_tag)::value;
        constexpr bool SAVE = decltype(save_tag)::value;
        const LayerDev& Ld = nd.layer[l];
        EpiFwd<T, ACT, SAVE> ep;
        ep.bias = theta_vec + Ld.vec_off;
        ep.H = Hbuf(l);
        ep.G = Gbuf(l);
        ep.ld = W;
        ep.part = nullptr;
        T* x0 = sv_x0;
        if (l == 0 && !x0 && use_x0(c)) x0 = reinterpret_cast<T*>(reinterpret_cast<float*>(wsT + 2 * ae) + part_elems(c, rs));
        if (l == 0 && x0) {
            const int64_t pieces = (int64_t)Mp * (x0_ld(c) / 8);
            k_gather_x<T><<<dim3((unsigned)((pieces + 255) / 256), P), 256, 0, s>>>(x, x0, O, x0_ld(c), M, Mp, rm);
        }
        if (l == 0 && use_x0(c)) {
            if constexpr (std::is_same<T, bf16_t>::value) {
                GemmArgs<T, SRC_KCONTIG, SRC_KCONTIG, EpiFwd<T, ACT, SAVE>, true, GEMM_NCH> g;
                g.a.base = x0; g.a.ld = O; g.a.rows = Mp; g.a.kdim = O; g.a.rm = rm;
                g.b.base = theta_mat + Ld.mat_off; g.b.ld = O; g.b.rows = W; g.b.kdim = O; g.b.rm = rm;
                g.a_pstride = (int64_t)Mp * O; g.b_pstride = nd.mat_len;
                g.epi = ep; g.e0_pstride = nd.vec_len; g.e1_pstride = (int64_t)Mp * W; g.e2_pstride = 0;
                run_gemm(c, 0, g, P, s);
            }
        } else if (l == 0 && first_fwd_narrow_ok(c)) {
            const int lds = (int)first_fwd_narrow_lds(c);
            static bool attr_set = false;
            if (!attr_set) {
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_first_fwd_narrow<T, ACT, SAVE>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
                attr_set = true;
            }
            GemmProf::Rec* r = prof_take(c, 0, 2.0 * M * (double)W * O * P);
            if (r) (void)hipEventRecord(r->a, s);
            k_first_fwd_narrow<T, ACT, SAVE><<<dim3((Mp + FN_ROWS - 1) / FN_ROWS, P), 256, lds, s>>>(
                x, theta_mat, theta_vec, nd.mat_len, nd.vec_len, Ld.mat_off, Ld.vec_off, O, W, M, Mp, rm, Hbuf(0), Gbuf(0));
            if (r) (void)hipEventRecord(r->b, s);
        } else if (l == 0) {
            auto launch = [&](auto fast) {
                constexpr bool F = decltype(fast)::value;
                GemmArgs<T, SRC_X_KCONTIG, SRC_KCONTIG, EpiFwd<T, ACT, SAVE>, F, GEMM_NCH> g;
                g.a.base = x; g.a.ld = O; g.a.rows = M; g.a.kdim = O; g.a.rm = rm;
                g.b.base = theta_mat + Ld.mat_off; g.b.ld = O; g.b.rows = W; g.b.kdim = O; g.b.rm = rm;
                g.a_pstride = 0; g.b_pstride = nd.mat_len;
                g.epi = ep; g.e0_pstride = nd.vec_len; g.e1_pstride = (int64_t)Mp * W; g.e2_pstride = 0;
                g.crows = Mp;
                run_gemm(c, 0, g, P, s);
            };
            if (O % VE == 0) launch(std::true_type{}); else launch(std::false_type{});
        } else {
            GemmArgs<T, SRC_KCONTIG, SRC_KCONTIG, EpiFwd<T, ACT, SAVE>, true, GEMM_NCH> g;
            g.a.base = Hbuf(l - 1); g.a.ld = W; g.a.rows = Mp; g.a.kdim = W; g.a.rm = rm;
            g.b.base = theta_mat + Ld.mat_off; g.b.ld = W; g.b.rows = W; g.b.kdim = W; g.b.rm = rm;
            g.a_pstride = (int64_t)Mp * W; g.b_pstride = nd.mat_len;
            g.epi = ep; g.e0_pstride = nd.vec_len; g.e1_pstride = (int64_t)Mp * W; g.e2_pstride = 0;
            run_gemm(c, 1, g, P, s);
        }
    };
    const FwdPlan plan = fwd_plan((int)sizeof(T), W, L, O, nd.out_dim, P, M, resident_slots() / 2,
                                  std::is_same<T, bf16_t>::value && fused_fwd_ok(c, nd, theta_mat));
    if (plan.rt > 0) {
        FwdArgs a;
        a.split = plan.split;
        fill_fwd_net(c, net, theta_mat, theta_vec, rs, out, saved_out, eps, act, logp, reinterpret_cast<char*>(sv),
                     reinterpret_cast<char*>(sv ? sv + ae : nullptr), reinterpret_cast<char*>(sv_x0), a.net);
        a.x = x; a.Mp = Mp; a.ldh = W; a.ldx = x0_ld(c); a.lstride = 2 * ae * (int64_t)sizeof(T);
        run_mlp_fwd(c, nd, a, plan.rt, sv != nullptr, s);
        return;
    }
    bool fused = false;
    if constexpr (std::is_same<T, bf16_t>::value) {
        if (fused_fwd_ok(c, nd, theta_mat)) {
            FusedFwdArgs a;
            a.x = x;
            a.x0 = sv_x0; a.ldx = x0_ld(c); a.Mp = Mp;
            a.theta_mat = theta_mat; a.theta_vec = theta_vec;
            a.Opad = (O + 63) & ~63;
            a.frag_len = fused_frag_len(c, net);
            a.mat_len = nd.mat_len; a.vec_len = nd.vec_len;
            for (int l = 0; l < L; ++l) { a.mat_off[l] = nd.layer[l].mat_off; a.vec_off[l] = nd.layer[l].vec_off; }
            {  // the matrices the kernel streams, once more in the order of its requests
                FragOrderArgs fo;
                fo.src = theta_mat; fo.dst = reinterpret_cast<bf16_t*>(ws); fo.mat_len = nd.mat_len; fo.L = L;
                fo.frag_len = a.frag_len;
                int g = 0;
                for (int l = 0; l < L; ++l) {
                    fo.mat_off[l] = nd.layer[l].mat_off;
                    fo.frag_off[l] = a.frag_off[l] = nd.layer[l].mat_off + (l > 0 ? (int64_t)W * (a.Opad - O) : 0);
                    fo.K[l] = l == 0 ? a.Opad : W;
                    fo.Ksrc[l] = l == 0 ? O : W;
                    fo.g0[l] = g;
                    g += (W / 64) * 2 * (fo.K[l] >> 6);
                }
                fo.g0[L] = g;
                k_theta_fragment_order<<<dim3(g, P), 256, 0, s>>>(fo);
                a.theta_frag = fo.dst;
            }
            a.H = sv;
            a.G = sv ? reinterpret_cast<gfix16_t*>(sv + ae) : nullptr;
            a.lstride = 2 * ae;
            a.L = L; a.O = O; a.M = M;
            a.tiles_m = (M + FF_ROWS - 1) / FF_ROWS;  // (128: covers Mp as well)
            a.n_tiles = a.tiles_m * P;
            const LayerDev& Lo = nd.layer[L];
            a.head_mat_off = Lo.mat_off; a.head_vec_off = Lo.vec_off; a.logsig_off = Lo.vec_off + Lo.d_out;
            a.out_dim = nd.out_dim;
            a.tanh_cols = (net == MORLAX_ACTOR && c->d.mean_tanh) ? c->d.act_dim : 0;
            a.adim = c->d.act_dim;
            a.sig_state = (net == MORLAX_ACTOR && c->d.sigma_state) ? 1 : 0;
            a.rm = rm; a.out = out; a.saved_out = saved_out; a.eps = eps; a.act = act; a.logp = logp;
            if (c->d.act == 0) {
                if (sv) launch_fused_fwd<0, true>(c, a, s); else launch_fused_fwd<0, false>(c, a, s);
            } else {
                if (sv) launch_fused_fwd<1, true>(c, a, s); else launch_fused_fwd<1, false>(c, a, s);
            }
            fused = true;
        }
    }
    for (int l = 0; l < L && !fused; ++l) {
        const bool save = sv != nullptr;
        if (c->d.act == 0) {
            if (save) layer(l, std::integral_constant<int, 0>{}, std::true_type{});
            else layer(l, std::integral_constant<int, 0>{}, std::false_type{});
        } else {
            if (save) layer(l, std::integral_constant<int, 1>{}, std::true_type{});
            else layer(l, std::integral_constant<int, 1>{}, std::false_type{});
        }
    }
    if (fused) return;  // the fused kernel applies the output layer as well
    const LayerDev& Lh = nd.layer[L];
    const int tanh_cols = (net == MORLAX_ACTOR && c->d.mean_tanh) ? c->d.act_dim : 0;
    const dim3 grid((M + 63) / 64, P);
    k_head_fwd<T><<<grid, 256, 0, s>>>(Hbuf(L - 1), theta_mat, theta_vec, nd.mat_len, nd.vec_len, Lh.mat_off,
                                       Lh.vec_off, W, nd.out_dim, M, Mp, rm, tanh_cols, out, saved_out, eps, act, logp,
                                       Lh.vec_off + Lh.d_out, c->d.act_dim,
                                       (net == MORLAX_ACTOR && c->d.sigma_state) ? 1 : 0);
}

template <typename T>
static void policy_bwd_t(const morlax_ctx* c, int net, const T* theta_mat, const float* theta_vec, const float* x,
                         const RowSel& rs, const void* saved, const float* dout, const float* dlogsig,
                         float* dtheta_mat, float* dtheta_vec, void* ws, hipStream_t s) {
    (void)theta_vec;
    const NetDev& nd = c->net[net];
    const int P = c->d.P, W = c->d.width, M = rs.M, L = c->d.n_hidden, O = c->d.obs_dim;
    const int Mp = pad_rows(rs);
    const int64_t ae = act_elems(c, rs);
    const RowMap rm = make_rowmap(c, rs);
    const T* sv = reinterpret_cast<const T*>(saved);
    T* wsT = reinterpret_cast<T*>(ws);
    auto Hbuf = [&](int l) { return sv + (int64_t)(2 * l) * ae; };
    typedef typename GradT<T>::type GT;
    auto Gbuf = [&](int l) { return reinterpret_cast<const GT*>(sv + (int64_t)(2 * l + 1) * ae); };
    auto dZbuf = [&](int l) { return wsT + (int64_t)(l & 1) * ae; };
    float* part = reinterpret_cast<float*>(wsT + 2 * ae);
    const BwdPart B = bwd_part(c, rs);
    const float* saved_out = reinterpret_cast<const float*>(sv + (int64_t)2 * L * ae);
    const LayerDev& Lh = nd.layer[L];
    const int n64 = (Mp + 63) / 64;
    BwdFinalArgs fin;
    fin.part = part; fin.dlogsig = dlogsig; fin.dmat = dtheta_mat; fin.dvec = dtheta_vec;
    fin.mat_len = nd.mat_len; fin.vec_len = nd.vec_len;
    fin.W = W; fin.L = L; fin.O = O; fin.OP = O <= 16 ? 16 : 32; fin.out_dim = nd.out_dim;
    fin.A = net == MORLAX_ACTOR && !c->d.sigma_state ? c->d.act_dim : 0;  // (a state-dependent log sigma is part of dout)
    fin.n_pb = n64; fin.first_ns = 0; fin.first = B.first; fin.pw = B.pw; fin.pb = B.pb;
    fin.mat_off[L] = Lh.mat_off; fin.vec_off[L] = Lh.vec_off; fin.logsig_off = Lh.vec_off + Lh.d_out;
    for (int l = 0; l < L; ++l) {
        fin.n_part[l] = n64;  // row blocks of whichever kernel produced the layer's dZ
        fin.S[l] = 1;
        fin.colsum[l] = B.colsum[l]; fin.split[l] = B.split[l];
        fin.mat_off[l] = nd.layer[l].mat_off; fin.vec_off[l] = nd.layer[l].vec_off;
        fin.n[l] = (int64_t)W * nd.layer[l].d_in;
    }
    {  // output layer
        HeadDz hz;
        hz.dout = dout; hz.saved_out = saved_out; hz.out_dim = nd.out_dim; hz.M = M; hz.rm = rm;
        hz.tanh_cols = (net == MORLAX_ACTOR && c->d.mean_tanh) ? c->d.act_dim : 0;
        const int ncol = (W + 127) / 128;
        // Up to one dW workgroup a CU, they start first: each walks a quarter of a preference's rows, and those of the last
        // preferences were at it long after the others had ended.  us a backward pass of one hidden layer, among the others and
        // first: 32 preferences x 8192 rows of 256 138 and 122, fp32, 16 x 8192 of 256 156 and 124, 8 x 3337 of 512 71 and 58; with
        // more of them there is too little else to run beside them (64 x 4096 of 512 234 and 238, 128 x 2048 229 and 239).
        const int n_dw = ncol * HB_SPLIT * P, n_front = n_dw <= resident_slots() / 2 ? n_dw : 0;
        const int per_rest = ncol * (n_front ? n64 : HB_SPLIT + n64);
        k_head_bwd<T><<<ncol * (HB_SPLIT + n64) * P, 256, 0, s>>>(hz, Hbuf(L - 1), theta_mat, nd.mat_len, Lh.mat_off, Gbuf(L - 1),
                                                                dZbuf(L - 1), part + B.pw, part + B.pb, part + B.colsum[L - 1], W, Mp,
                                                                n_front, per_rest, row_div(ncol * HB_SPLIT), row_div(per_rest));
    }
    for (int l = L - 1; l >= 0; --l) {
        const LayerDev& Ld = nd.layer[l];
        // dW_l = dZ_l^T in: `in` the layer's compact input, [P][Mp][ld]
        auto weight_grad = [&](int kind, const T* in, int ld) {
            GemmArgs<T, SRC_KSTRIDED, SRC_KSTRIDED, EpiDw, true, GEMM_NCH> g;
            g.a.base = dZbuf(l); g.a.ld = W; g.a.rows = W; g.a.kdim = Mp; g.a.rm = rm;
            g.b.base = in; g.b.ld = ld; g.b.rows = ld; g.b.kdim = Mp; g.b.rm = rm;
            g.a_pstride = (int64_t)Mp * W; g.b_pstride = (int64_t)Mp * ld;
            g.ccols = Ld.d_in;
            g.epi.dW = dtheta_mat + Ld.mat_off; g.epi.ld = Ld.d_in; g.epi.part = nullptr;
            g.e0_pstride = nd.mat_len; g.e1_pstride = 0; g.e2_pstride = 0;
            const int S = dw_split(c, M, l, false);
            if (S > 1) {
                g.range = dw_range(rs, S);
                g.ranges = (Mp + g.range - 1) / g.range;
                g.epi.dW = part + B.split[l]; g.e0_pstride = fin.n[l];
                fin.S[l] = g.ranges;
            }
            run_gemm(c, kind, g, P * g.ranges, s);
        };
        if (l > 0) {
            weight_grad(3, Hbuf(l - 1), W);
            GemmArgs<T, SRC_KCONTIG, SRC_KSTRIDED, EpiDx<T>, true, GEMM_NCH> h;
            h.a.base = dZbuf(l); h.a.ld = W; h.a.rows = Mp; h.a.kdim = W; h.a.rm = rm;
            h.b.base = theta_mat + Ld.mat_off; h.b.ld = W; h.b.rows = W; h.b.kdim = W; h.b.rm = rm;
            h.a_pstride = (int64_t)Mp * W; h.b_pstride = nd.mat_len;
            h.epi.G = Gbuf(l - 1); h.epi.dZ = dZbuf(l - 1); h.epi.ld = W; h.epi.part = part + B.colsum[l - 1];
            h.e0_pstride = (int64_t)Mp * W; h.e1_pstride = 0; h.e2_pstride = 0;
            run_gemm(c, 2, h, P, s);
            fin.n_part[l - 1] = h.tiles_m;  // row tiles of the kernel that ran (128 or 256 rows)
        } else if (first_skinny(c)) {
            const int ns = first_split(c, rs);
            GemmProf::Rec* r = prof_take(c, 4, 2.0 * W * (double)O * M * P);
            if (r) (void)hipEventRecord(r->a, s);
            const dim3 grid((W + 127) / 128, ns, P);
            if (fin.OP == 16) k_first_bwd_dw<T, 1><<<grid, 256, 0, s>>>(x, dZbuf(0), part + B.first, O, W, M, Mp, ns, rm);
            else k_first_bwd_dw<T, 2><<<grid, 256, 0, s>>>(x, dZbuf(0), part + B.first, O, W, M, Mp, ns, rm);
            if (r) (void)hipEventRecord(r->b, s);
            fin.first_ns = ns;
        } else {
            weight_grad(4, reinterpret_cast<const T*>(reinterpret_cast<const char*>(sv) + saved_x0_off(c, rs)), x0_ld(c));
        }
    }
    int b = L * ((W + 31) / 32);
    fin.b_head = b;
    b += (nd.out_dim * W + 255) / 256;
    for (int l = 0; l < L; ++l) {
        fin.b_split[l] = b;
        if (fin.S[l] > 1) b += (int)((fin.n[l] / 4 + 255) / 256);
    }
    fin.b_first = b;
    if (fin.first_ns > 0) b += (W + 31) / 32 * ((O + 7) / 8);
    k_bwd_final<<<dim3(b, P), 256, 0, s>>>(fin);
}

void launch_policy_fwd(const morlax_ctx* c, int net, const void* theta_mat, const float* theta_vec,
                       const float* x, const RowSel& rs, float* out, const float* eps, float* act,
                       float* logp, void* saved, void* ws, hipStream_t s) {
    if (c->d.wdtype == 1)
        policy_fwd_t<bf16_t>(c, net, (const bf16_t*)theta_mat, theta_vec, x, rs, out, eps, act, logp, saved, ws, s);
    else
        policy_fwd_t<float>(c, net, (const float*)theta_mat, theta_vec, x, rs, out, eps, act, logp, saved, ws, s);
}

void launch_policy_bwd(const morlax_ctx* c, int net, const void* theta_mat, const float* theta_vec,
                       const float* x, const RowSel& rs, const void* saved, const float* dout,
                       const float* dlogsig, float* dtheta_mat, float* dtheta_vec, void* ws,
                       hipStream_t s) {
    if (c->d.wdtype == 1)
        policy_bwd_t<bf16_t>(c, net, (const bf16_t*)theta_mat, theta_vec, x, rs, saved, dout, dlogsig, dtheta_mat,
                             dtheta_vec, ws, s);
    else
        policy_bwd_t<float>(c, net, (const float*)theta_mat, theta_vec, x, rs, saved, dout, dlogsig, dtheta_mat,
                            dtheta_vec, ws, s);
}
