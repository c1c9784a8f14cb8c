// Device-side pieces shared by the FP16/BF16 matrix-core kernels: operand types,
// the matrix instruction, packing of accumulators into the next operand, and the
// encoding of a record into an LDS row by eight lanes.
#pragma once

#include "encode_impl.h"
#include "nrc_internal.h"

namespace nrc {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Vec8;
template <> struct Vec8<_Float16> { typedef f16x8 type; };
template <> struct Vec8<__bf16> { typedef bf16x8 type; };

__device__ inline f32x4 mfma(f16x8 a, f16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ inline f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// x r rounded to the operand type.  FP16: once, by the mixed multiply-add; left
// to the compiler the product is rounded to FP32 first in some kernels and not in
// others, and a record's gradient would depend on the kernel its batch takes.
template <typename T> __device__ inline T mul_to(float x, float r) {
    if constexpr (__is_same(T, _Float16)) {
        unsigned int d = 0;
        asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "+v"(d) : "v"(x), "v"(r));
        return __builtin_bit_cast(_Float16, (unsigned short)d);
    } else {
        return (T)(x * r);
    }
}

template <typename V> __device__ inline V zero8() {
    V v;
    #pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0;
    return v;
}

// Two accumulator blocks (features 4g..4g+3 and 16+4g..16+4g+3 of a chunk)
// -> one B operand in chained order.
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename T, typename V> __device__ inline V pack8(f32x4 lo, f32x4 hi) {
    if constexpr (sizeof(T) == 2 && !__is_same(T, _Float16)) {
        // BF16: one v_cvt_pk_bf16_f32 per pair (the generic vector conversion
        // is split into single conversions and byte permutes)
        u32x4 r;
        r[0] = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{lo[0], lo[1]}, bf16x2));
        r[1] = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{lo[2], lo[3]}, bf16x2));
        r[2] = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{hi[0], hi[1]}, bf16x2));
        r[3] = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{hi[2], hi[3]}, bf16x2));
        return __builtin_bit_cast(V, r);
    } else {
        const f32x8 f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_convertvector(f, V);
    }
}

typedef short s16x8 __attribute__((ext_vector_type(8)));

// ReLU on a packed FP16/BF16 operand: a negative value has its sign bit set,
// so as a signed 16-bit integer it is negative and max(., 0) maps it to +0;
// non-negative values are unchanged.  Rounding preserves sign, so
// relu(round(x)) == round(relu(x)).
template <typename V> __device__ inline V relu_packed(V v) {
    s16x8 i = __builtin_bit_cast(s16x8, v);
    i = __builtin_elementwise_max(i, (s16x8)(0));
    return __builtin_bit_cast(V, i);
}

// Reflectance factor alpha + beta (Sec. 5) of record ln from the B operand
// holding input features 32..63 in natural order (lane 16g + ln: features
// 32 + 8g .. 32 + 8g + 7); valid in lanes 0..15, 1 when fcol == 0.  Config
// preset: diffuse 53..55 sit in lane 32 + ln, slots 5..7, and specular 56..58
// in lane 48 + ln, slots 0..2; paper presets: both in lane 48 + ln, slots 0..5.
template <typename V>
__device__ inline void reflectance_operand(const V& b1, int fcol, int ln, float (&r)[3]) {
    if (fcol == kAlbedoColConfig) {
        #pragma unroll
        for (int c = 0; c < 3; ++c)
            r[c] = __shfl((float)b1[5 + c], 32 + ln, 64) + __shfl((float)b1[c], 48 + ln, 64);
    } else if (fcol == kAlbedoColPaper) {
        #pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = __shfl((float)b1[c] + (float)b1[3 + c], 48 + ln, 64);
    } else {
        r[0] = r[1] = r[2] = 1.0f;
    }
}

// Features 8q .. 8q + 7 of f, rounded to T, into an LDS row.
template <typename T>
__device__ inline void store8(T* dst, const float* f, int q) {
    using V = typename Vec8<T>::type;
    const f32x4 lo = f32x4{f[8 * q], f[8 * q + 1], f[8 * q + 2], f[8 * q + 3]};
    const f32x4 hi = f32x4{f[8 * q + 4], f[8 * q + 5], f[8 * q + 6], f[8 * q + 7]};
    *reinterpret_cast<V*>(dst + 8 * q) = pack8<T, V>(lo, hi);
}

// A record at rr (14 or 16 floats) encoded into the LDS row h0 by eight lanes, two
// of each of four lane groups: first (half 0) the frequency encodings, position
// coordinate g per group, then (half 1) the one-blob of angle g and a quarter of
// the rest.  Both halves of a record run at once, in different waves, and neither
// diverges far.  valid = false: zeros.  The same arithmetic as encode_part.  Feature
// k goes to k ^ key (a multiple of 4).
template <typename T, int PRESET, int LAYOUT>
__device__ inline void encode_half(const float* __restrict__ rr, T* h0, int key, int half, int g, bool valid) {
    constexpr bool paper = PRESET != NRC_PRESET_CONFIG, gauss = PRESET == NRC_PRESET_PAPER_GAUSS;
    if (half == 0) {
        if (g < 3) {
            float x[1] = {valid ? rr[g] : 0.0f}, f[64];
            encode_part<PRESET, LAYOUT, 0>(x, f);
            #pragma unroll
            for (int k = 0; k < 12; ++k) f[k] = valid ? f[k] : 0.0f;
            #pragma unroll
            for (int q = 0; q < 3; ++q) store4<T>(h0 + ((12 * g + 4 * q) ^ key), f + 4 * q);
        }
        return;
    }
    const float* rest = rr + (LAYOUT == NRC_RAW14 ? 7 : 9);
    float v[7], s = 0.0f;
    #pragma unroll
    for (int j = 0; j < 7; ++j) v[j] = valid ? rest[j] : 0.0f;
    if (LAYOUT == NRC_RAW14) {
        if (valid) s = rr[3 + g];
    } else if (valid) {
        const float* d = rr + 3 + 3 * (g >> 1);
        float u, w;
        sph(d[0], d[1], d[2], u, w);
        s = g & 1 ? w : u;
    }
    float e[4];
    if (gauss) one_blob4_gauss(s, e); else one_blob4(s, e);
    #pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = valid ? e[k] : 0.0f;
    store4<T>(h0 + ((36 + 4 * g) ^ key), e);
    if (g == 3) return;
    if (paper) {
        const float one = valid ? 1.0f : 0.0f;
        if (g == 0) {
            if (gauss) one_blob4_gauss(1.0f - expf(-v[0]), e); else one_blob4(1.0f - expf(-v[0]), e);
            #pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = valid ? e[k] : 0.0f;
        } else {
            e[0] = g == 1 ? v[1] : v[5];
            e[1] = g == 1 ? v[2] : v[6];
            e[2] = g == 1 ? v[3] : one;
            e[3] = g == 1 ? v[4] : one;
        }
    } else {
        e[0] = g == 0 ? v[0] : g == 1 ? v[4] : 0.0f;
        e[1] = g == 0 ? v[1] : g == 1 ? v[5] : 0.0f;
        e[2] = g == 0 ? v[2] : g == 1 ? v[6] : 0.0f;
        e[3] = g == 0 ? v[3] : 0.0f;
    }
    store4<T>(h0 + ((52 + 4 * g) ^ key), e);
}

}  // namespace
}  // namespace nrc
