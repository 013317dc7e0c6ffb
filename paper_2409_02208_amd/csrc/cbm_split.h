// A 32-bit value as three bf16 values that add up to it exactly, for matrix-core products that keep 32-bit operands (device code).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// x minus the low (high) half of a pair of bf16 values: one instruction, and exact where the half is x's leading bits.
// `minus_low` = (-1, 0) comes from a register: as an inline constant -1.0 would stand for (0, -1).
__device__ __forceinline__ float less(float x, uint32_t pair, uint32_t which) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, which), x, false);
}
__device__ __forceinline__ uint32_t high_halves(float x0, float x1) {
    return __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
}
// The 24 significant bits of a value as three bf16 values (8 + 8 + 8 bits, by truncation, so nothing is rounded and nothing
// overflows): x = h + m + l exactly.  Two values at a time, packed as an operand wants them.
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t minus_low, uint32_t& h, uint32_t& m, uint32_t& l) {
    const uint32_t minus_high = 0xbf800000u;
    h = high_halves(x0, x1);
    x0 = less(x0, h, minus_low);
    x1 = less(x1, h, minus_high);
    m = high_halves(x0, x1);
    x0 = less(x0, m, minus_low);
    x1 = less(x1, m, minus_high);
    l = high_halves(x0, x1);
}
// The same with every part rounded to the nearest: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|, of either sign, and still x = h + m + l exactly
// (what rounding leaves of x fits the next part).  Values that round up to infinity have no parts: their remainders are not
// finite, nor is any sum with them.
__device__ __forceinline__ uint32_t nearest_pair(float x0, float x1) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){x0, x1}, bf16x2));
}
__device__ __forceinline__ void split_pair_nearest(float x0, float x1, uint32_t minus_low, uint32_t& h, uint32_t& m, uint32_t& l) {
    const uint32_t minus_high = 0xbf800000u;
    h = nearest_pair(x0, x1);
    x0 = less(x0, h, minus_low);
    x1 = less(x1, h, minus_high);
    m = nearest_pair(x0, x1);
    x0 = less(x0, m, minus_low);
    x1 = less(x1, m, minus_high);
    l = nearest_pair(x0, x1);
}
