// Device helpers shared by the target-network kernels: row map, packing, MFMA wrappers, activations.
#pragma once

#include <type_traits>

#include "morlax_internal.h"
#include "numeric.h"

#define OUT_PITCH 16       // floats per row of the saved head output

struct RowMap {  // compact row m of preference p -> row of a time-major tensor
    int32_t t0, j0, j_cnt, N, n_g;
    RowDiv by;  // of j_cnt (a division by the compiler is some twenty instructions for every row a lane looks up)
    __device__ inline int64_t row(int p, int m) const {
        const int t = (int)by.quotient((uint32_t)m);
        return (int64_t)(t0 + t) * N + (int64_t)p * n_g + j0 + (m - t * j_cnt);
    }
};

template <typename T> struct Elems { static constexpr int VE = 16 / sizeof(T); };

// (converted as a pair: one instruction; two conversions and a merge otherwise)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t{a, b}), bf16x2_t));
}

template <typename T> __device__ inline uint4 pack_chunk(const float* v);  // 16 bytes of GEMM inputs
template <> __device__ inline uint4 pack_chunk<float>(const float* v) {
    return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
}
template <> __device__ inline uint4 pack_chunk<bf16_t>(const float* v) {
    return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
}

template <typename T> struct Mma32;
template <> struct Mma32<bf16_t> {
    static __device__ inline void run(const uint4& a, const uint4& b, float16_t& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                    0, 0, 0);
    }
};
constexpr float kBf16Largest = 0x1.fep127f;
// An fp32 value as the sum of three bf16 values, each the nearest to what those before it leave: 24 bits exactly, down to
// some 1e-30; below, the smallest part and then the middle one are subnormal, and the matrix instructions take those for zero (a
// backward pass whose largest dW is 5e-30, 5e-33, 3e-34, 1e-36: off by 1e-9, 2e-7, 4e-6, 9e-4 of itself; on the fp32 instructions
// by 1e-7 at the last).  A product
// of two such values is nine products of parts; the three smallest (2^-24 of it and less) are dropped, and the other six run on
// the bf16 matrix instructions, sixteen times as fast as the fp32 ones.  Sums of the five smaller ones are kept apart from those
// of the leading parts, which then take one rounding per sixteen products.  Against 64 bits, normal operands: 3.0e-8 of the
// result for 16 products, 9.3e-8 for 256, 6.0e-7 for 8192, where the fp32 instructions give 7.0e-8, 2.9e-7 and 1.7e-6 (all nine
// products: the same figures; all six in one accumulator: 3.2e-8, 2.5e-7, 1.5e-6).
// An infinite value leaves undefined smaller parts, and so does a finite one that rounds to an infinite bf16 value (beyond 3.396e38,
// within 2^-9 of the largest); a leading product within as much of it may overflow where the exact one does not.  any_undefined
// tells, and the block is multiplied again by the fp32 instructions.  BOUNDED: the leading part stops at the largest bf16 value, so
// that the parts of every finite value add up to it; an infinite one's second part is infinite.
template <bool BOUNDED = false>
__device__ inline void split3(const uint4& u, uint2 part[3]) {
    float v[4] = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = BOUNDED && q == 0 ? __builtin_amdgcn_fmed3f(v[e], -kBf16Largest, kBf16Largest) : v[e];
        part[q] = make_uint2(pack2(t[0], t[1]), pack2(t[2], t[3]));
        if (q < 2) {
            v[0] -= __uint_as_float(part[q].x << 16); v[1] -= __uint_as_float(part[q].x & 0xffff0000u);
            v[2] -= __uint_as_float(part[q].y << 16); v[3] -= __uint_as_float(part[q].y & 0xffff0000u);
        }
    }
}
template <bool BOUNDED = false>
__device__ inline void split3(const float (&v)[8], uint4 (&part)[3]) {
    uint2 lo[3], hi[3];
    split3<BOUNDED>(make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])), lo);
    split3<BOUNDED>(make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])), hi);
#pragma unroll
    for (int q = 0; q < 3; ++q) part[q] = make_uint4(lo[q].x, lo[q].y, hi[q].x, hi[q].y);
}
// term t = 0 .. 5 of a product of split operands, smallest first
__device__ inline void split_mma(int t, const uint4 (&a)[3], const uint4 (&b)[3], float16_t& acc, float16_t& low) {
    const int i = t == 0 ? 0 : t == 1 ? 2 : t == 2 ? 1 : t == 3 ? 0 : t == 4 ? 1 : 0;
    const int j = t == 0 ? 2 : t == 1 ? 0 : t == 2 ? 1 : t == 3 ? 1 : 0;
    Mma32<bf16_t>::run(a[i], b[j], t == 5 ? acc : low);
}
// does a wave hold an undefined or infinite sum (or sums of one lane that add up to one: multiplied again for nothing)
__device__ inline bool any_undefined(float t) { return __any(!(__builtin_fabsf(t) < __builtin_inff())); }
__device__ inline bool any_undefined(const float16_t& v) {
    float t = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) t += v[e];
    return any_undefined(t);
}

__device__ inline float chunk_f32(const uint4& u, int e) {  // e a compile-time constant after unrolling
    return __uint_as_float(e == 0 ? u.x : e == 1 ? u.y : e == 2 ? u.z : u.w);
}

template <typename T> struct Mma16;
template <> struct Mma16<bf16_t> {
    static __device__ inline void run(const uint4& a, const uint4& b, float4_t& c) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                    0, 0, 0);
    }
};
template <> struct Mma16<float> {
    static __device__ inline void run(const uint4& a, const uint4& b, float4_t& c) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};

// h = act(z) and g = act'(z) of a network with GEMM inputs of type T.  SiLU uses the hardware exp2 / reciprocal
// approximations (about 1 ulp each): s = 1 / (1 + e^-z), h = z s, g = s (1 + z - h).  In bf16 networks every kernel that
// may serve a layer rounds g alike: FUSED with h = z s inside a fused multiply-add, else without.  (Another rounding of g
// moves the gradients by 4e-5, which six Adam steps, whose normalised step turns the sign of a gradient near zero into a
// whole step, turned into 0.12.)  tanh is the library's routine.
template <typename T, int ACT, bool FUSED>
__device__ inline void act_pair(float z, float& h, float& g) {
    if (ACT == 0) {
        h = tanhf(z);
        g = 1.f - h * h;
    } else {
        const float e = __expf(-z);
        const float s = __builtin_amdgcn_rcpf(1.f + e);
        h = z * s;
        if (sizeof(T) == 4) {
            g = s * (1.f + z - h);
        } else if (FUSED) {
            g = s * __builtin_fmaf(-z, s, 1.f + z);
        } else {
#pragma clang fp contract(off)
            const float z1 = 1.f + z, d = z1 - h;
            g = s * d;
        }
    }
}

// eight consecutive elements of type T / of the saved-derivative type: packing and 16-byte accesses
struct Pack8 { uint4 lo, hi; };  // bf16 / fixed point use lo only; fp32 uses both
__device__ inline Pack8 pack8(const float v[8], const float*) {
    Pack8 r;
    r.lo = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
    r.hi = make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7]));
    return r;
}
__device__ inline Pack8 pack8(const float v[8], const bf16_t*) {
    Pack8 r;
    r.lo = pack_chunk<bf16_t>(v);
    r.hi = make_uint4(0, 0, 0, 0);
    return r;
}
__device__ inline Pack8 pack8(const float v[8], const gfix16_t*) {
    // round(v / step + 1/8 / step); values are in (-0.125, 1.125) so the conversion cannot overflow
    uint32_t q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = (uint32_t)(v[i] * (1.0f / GFIX_STEP) + (0.125f / GFIX_STEP + 0.5f));
    Pack8 r;
    r.lo = make_uint4(q[0] | (q[1] << 16), q[2] | (q[3] << 16), q[4] | (q[5] << 16), q[6] | (q[7] << 16));
    r.hi = make_uint4(0, 0, 0, 0);
    return r;
}
__device__ inline void put8(float* dst, const Pack8& pk) {
    reinterpret_cast<uint4*>(dst)[0] = pk.lo;
    reinterpret_cast<uint4*>(dst)[1] = pk.hi;
}
__device__ inline void put8(bf16_t* dst, const Pack8& pk) { *reinterpret_cast<uint4*>(dst) = pk.lo; }
__device__ inline void put8(gfix16_t* dst, const Pack8& pk) { *reinterpret_cast<uint4*>(dst) = pk.lo; }
__device__ inline void get8(const float* src, float v[8]) {
    const float4 a = reinterpret_cast<const float4*>(src)[0], b = reinterpret_cast<const float4*>(src)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ inline void unpack8(const uint4& u, float v[8]) {  // eight fixed-point derivatives
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = (float)(w[i] & 0xffffu) * GFIX_STEP - 0.125f;
        v[2 * i + 1] = (float)(w[i] >> 16) * GFIX_STEP - 0.125f;
    }
}
__device__ inline void get8(const gfix16_t* src, float v[8]) {
    const uint4 u = *reinterpret_cast<const uint4*>(src);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = (float)(w[i] & 0xffffu) * GFIX_STEP - 0.125f;
        v[2 * i + 1] = (float)(w[i] >> 16) * GFIX_STEP - 0.125f;
    }
}

// Logical tile id so that consecutive ids run on the same XCD (workgroups are dealt round-robin to
// the 8 XCDs by hardware id): the tiles of one preference then share that XCD's L2 copy of W(p).
__device__ inline int xcd_remap(int bid, int nb) {
    const int q = nb / 8, rem = nb % 8, x = bid % 8, pos = bid / 8;
    return x * q + (x < rem ? x : rem) + pos;
}
