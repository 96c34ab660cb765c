// fp32 values as two scaled fp16 terms, x s = h0 + h1 / kHalfLow (kernels_gemm_half.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

constexpr float kHalfLow = 2048.f;     // scale of the second term
constexpr int kHalfTop = 14;           // exponent that the largest weight of a column is brought to when its copy is made

// Two fp32 values, already scaled, as their two fp16 terms (the first value in the low half).
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    const halfx2 h = __builtin_convertvector((floatx2{x0, x1}), halfx2);
    const halfx2 l = {_Float16(__builtin_fmaf(float(h[0]), -kHalfLow, x0 * kHalfLow)), _Float16(__builtin_fmaf(float(h[1]), -kHalfLow, x1 * kHalfLow))};
    hi = __builtin_bit_cast(uint32_t, h), lo = __builtin_bit_cast(uint32_t, l);
}

// And what the second terms leave, at their scale: x s = h0 + (h1 + h2) / kHalfLow.
__device__ __forceinline__ uint32_t third_pair(float x0, float x1, uint32_t hi, uint32_t lo) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    const halfx2 h = __builtin_bit_cast(halfx2, hi), l = __builtin_bit_cast(halfx2, lo);
    const floatx2 r = {__builtin_fmaf(float(h[0]), -kHalfLow, x0 * kHalfLow) - float(l[0]), __builtin_fmaf(float(h[1]), -kHalfLow, x1 * kHalfLow) - float(l[1])};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(r, halfx2));
}

// Largest value of a group of 4, 8 or 16 consecutive lanes, in all of them.
template <int CTRL>
__device__ __forceinline__ float max_moved(float x) {
    return fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, int(__float_as_uint(x)), CTRL, 0xF, 0xF, false)));
}
template <int LANES>
__device__ __forceinline__ float largest_of_lanes(float x) {
    static_assert(LANES == 4 || LANES == 8 || LANES == 16, "a row of lanes or a part of it");
    x = max_moved<0x4E>(max_moved<0xB1>(x));           // quad_perm: lane xor 1, lane xor 2
    if (LANES >= 8) x = max_moved<0x141>(x);           // row_half_mirror
    return LANES == 16 ? max_moved<0x128>(x) : x;      // row_ror 8
}

// Exponent of the scale that brings `largest` (>= 0; zero and denormals count as the smallest normal number) to [2^target,
// 2^(target + 1)), as far as the scale is a normal number.
__device__ __forceinline__ int scale_exponent(float largest, int target) { return min(target + 127 - int(__float_as_uint(largest) >> 23), 126); }
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float(uint32_t(e + 127) << 23); }      // -126 <= e <= 127
