// Device helpers shared by the operand-preparation kernels and the single-launch
// short-sequence kernel: the key order inside a block image, the per-channel absmax of V
// and the 8-bit quantiser psi of Eq. 7.
#pragma once

#include "binattn_internal.h"

namespace binattn {

typedef unsigned u4 __attribute__((ext_vector_type(4)));

// Eq. 5 for 8 bf16 values: bit i = (x_i >= 0) under IEEE rules (-0.0 -> 1, NaN -> 0, Sec. 3);
// adds their magnitudes to asum.
__device__ __forceinline__ unsigned sign_bits8_abs(u4 w, float &asum) {
    unsigned bits = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(w[i] << 16);
        const float hi = __uint_as_float(w[i] & 0xffff0000u);
        bits |= (lo >= 0.0f ? 1u : 0u) << (2 * i);
        bits |= (hi >= 0.0f ? 1u : 0u) << (2 * i + 1);
        asum += fabsf(lo) + fabsf(hi);
    }
    return bits;
}

// FP4 codes of +-1 of 8 bf16 values (nibble order of fp4_pm1_from_bits8) without going through
// sign bits; adds their magnitudes to asum.  Subtracting 1 with unsigned saturation from a
// 16-bit pattern leaves its top bit set exactly where the value is negative (-0.0, 0x8000,
// becomes 0x7FFF; 0 stays 0): one packed instruction per two values.  Only a NaN with the sign
// bit clear comes out wrong (+1 instead of -1): it turns asum into NaN, and the callers then
// redo their words with fp4_pm1_exact.  11 + 16 instructions per 8 values instead of 48.
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned neg_flags(unsigned w) {  // bits 15 and 31
    return __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(us2, w), us2{1, 1}));
}
__device__ __forceinline__ unsigned fp4_pm1_abs(u4 w, float &asum) {
    constexpr unsigned M = 0x80008000u;
    const unsigned hi = (neg_flags(w[3]) & M) | ((neg_flags(w[2]) >> 4) & (M >> 4));
    const unsigned lo = (neg_flags(w[1]) & M) | ((neg_flags(w[0]) >> 4) & (M >> 4));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        asum += fabsf(__uint_as_float(w[i] << 16)) + fabsf(__uint_as_float(w[i] & 0xffff0000u));
    }
    return (hi | (lo >> 8)) | 0x22222222u;
}
__device__ __forceinline__ unsigned fp4_pm1_exact(u4 w) {
    float unused = 0.0f;
    return fp4_pm1_from_bits8(sign_bits8_abs(w, unused));
}

// Row position inside a key block <-> key offset.  The fused kernel's lane
// (g = lane / 32) holds, for MFMA tile t and accumulator register r, the key
// j0 + 32 t + 16 g + r; the MFMA puts accumulator register r of lane group g
// at tile row m = 8 (r / 4) + 4 g + (r % 4).  Rows are stored at position
// 32 t + m so that the A operand reads consecutive LDS rows.
__device__ __forceinline__ int key_of_position(int pos) {
    const int t = pos >> 5, m = pos & 31;
    const int g = (m >> 2) & 1;
    const int r = ((m >> 3) << 2) | (m & 3);
    return 32 * t + 16 * g + r;
}
// Inverse of key_of_position: where key offset o (0 <= o < BV) sits in a block image.
__device__ __forceinline__ int position_of_key(int o) {
    return (o & 0x63) | ((o & 0x0C) << 1) | ((o >> 2) & 4);
}
// Single-launch forms: the key (offset inside its block) that the i-th group of a block's chunks belongs
// to.  Which keys a thread adds |k| of, and in which order, decides the last bits of the abs-mean:
// this assignment is part of the results and does not follow the layout of the image.
__device__ __forceinline__ int key_of_chunk(int i) {
    return ((i & 4) << 4) | ((i >> 1) & 0x3C) | (i & 3);  // 64 ((m >> 2) & 1) + 16 t + 4 (m >> 3) + (m & 3), i = 32 t + m
}

__device__ __forceinline__ void unpack8(u4 w, float f[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

// Running absmax of 8 bf16 values per lane on their bit patterns: with the sign bit
// cleared, bf16 magnitudes order like 16-bit unsigned integers (two values per instruction).
__device__ __forceinline__ void absmax_acc(unsigned m[4], u4 w) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const us2 a = __builtin_bit_cast(us2, m[i]);
        const us2 b = __builtin_bit_cast(us2, w[i] & 0x7FFF7FFFu);
        m[i] = __builtin_bit_cast(unsigned, __builtin_elementwise_max(a, b));
    }
}
__device__ __forceinline__ void absmax_floats(const unsigned m[4], float f[8]) {
    unpack8(u4{m[0], m[1], m[2], m[3]}, f);
}

// Eq. 7 scale: absmax / 127 (IEEE fp32 division); 1 for an all-zero channel.
__device__ __forceinline__ float delta_of_absmax(float a) {
    return (a == 0.0f) ? 1.0f : __fdiv_rn(a, 127.0f);
}

// Eq. 7: code = round-to-nearest-even(y), clamped to [-127, 127], with y = fp32(v / delta) and
// delta = fp32(a / 127), both IEEE divisions.  Fast form: one FMA, fma(v, r, 1.5 * 2^23), which
// rounds the exact product v r to an integer (ties to even) and leaves its two's complement
// code in the low byte.  It gives the code of y for EVERY bf16 v with |v| <= a because bf16
// significands are 8-bit integers: with v = V 2^s, a = A 2^t (128 <= A <= 255, e = t - s >= 0)
// the real quotient 127 v / a differs from a half-integer (2 k + 1) / 2, relative to it, by
// |254 V - (2 k + 1) A 2^e| / ((2 k + 1) A 2^e): either 0 or more than 2^-16, since the
// denominator is then about 254 V < 2^16.  y and v r (r within 2^-20 of 127 / a) both stay on
// the quotient's side of every half-integer it does not hit.  It hits one only if
//   * 127 divides A, i.e. A = 254: delta is a power of two, r = 1 / delta is exact, and both
//     forms see the same exact tie; or
//   * 127 divides 2 k + 1, i.e. 2 k + 1 = 127: v = a / 2 exactly, one magnitude per channel.
//     r is moved by 2^-21 to the side on which y rounds there (quant_consts).
// A channel whose a is outside [2^-100, 2^100] (bf16 denormals, 1 / delta out of range) gets
// r = 0 and its codes from the division.  The form before it (two FMAs with bracketing
// reciprocals, compared, the division where they differ) took 5 instructions per value
// instead of 2 and was two thirds of the V phase of the single-launch kernel.
constexpr float QMAGIC = 12582912.0f;  // 1.5 * 2^23
__device__ __forceinline__ float quant_exact(float v, float delta) {
    if (delta == INFINITY) return QMAGIC;  // an infinity in the channel: code 0 (0 x inf, not a number, comes out)
    return fminf(fmaxf(rintf(__fdiv_rn(v, delta)), -127.0f), 127.0f) + QMAGIC;
}
// The multipliers of 8 consecutive channels, read from LDS with 16-byte loads up front (the
// array must be 16-byte aligned).
struct QuantConsts8 {
    float r[8];
    bool exact;  // some channel takes the division
};
__device__ __forceinline__ QuantConsts8 load_quant_consts8(const float *srcp, int c) {
    QuantConsts8 k;
    const float4 *a = reinterpret_cast<const float4 *>(srcp + 8 * c);
    const float4 x = a[0], y = a[1];
    k.r[0] = x.x; k.r[1] = x.y; k.r[2] = x.z; k.r[3] = x.w;
    k.r[4] = y.x; k.r[5] = y.y; k.r[6] = y.z; k.r[7] = y.w;
    float lo = k.r[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) lo = fminf(lo, k.r[i]);
    k.exact = lo == 0.0f;
    return k;
}
// codes of 4 tokens x 8 channels (w[k]: token k), one dword per channel, token k in byte k.
// sdelta: the head's scales (LDS), read only where a channel needs the division.
__device__ __forceinline__ void quant_quad(const u4 w[4], const QuantConsts8 &kc, const float *sdelta, int c,
                                           unsigned packed[8]) {
    float f[4][8];
#pragma unroll
    for (int k = 0; k < 4; ++k) unpack8(w[k], f[k]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = fmaf(f[k][i], kc.r[i], QMAGIC);
        const unsigned b01 = __builtin_amdgcn_perm(__float_as_uint(s[1]), __float_as_uint(s[0]), 0x0c0c0400u);
        const unsigned b23 = __builtin_amdgcn_perm(__float_as_uint(s[3]), __float_as_uint(s[2]), 0x0c0c0400u);
        packed[i] = b01 | (b23 << 16);
    }
    if (kc.exact) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (kc.r[i] != 0.0f) continue;
            const float dl = sdelta[8 * c + i];
            unsigned q = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) q |= (__float_as_uint(quant_exact(f[k][i], dl)) & 0xFFu) << (8 * k);
            packed[i] = q;
        }
    }
}
// delta and the quantiser's multiplier of a channel from its absmax (a bf16 value)
__device__ __forceinline__ void quant_consts(float a, float *dl, float *r_out) {
    *dl = delta_of_absmax(a);
    const float r = __fdiv_rn(1.0f, *dl);
    if (a == 0.0f || (__float_as_uint(a) & 0x007F0000u) == 0x007E0000u) {  // delta 1 or a power of two
        *r_out = r;
    } else {
        // the code of v = a / 2 decides the side (y = 63.5 is a tie and goes to 64)
        const bool up = rintf(__fdiv_rn(0.5f * a, *dl)) == 64.0f;
        *r_out = __fmul_rn(r, up ? 1.0f + 0x1p-21f : 1.0f - 0x1p-21f);
    }
    if (a != 0.0f && !(a >= 0x1p-100f && a <= 0x1p100f)) *r_out = 0.0f;
}

}  // namespace binattn
