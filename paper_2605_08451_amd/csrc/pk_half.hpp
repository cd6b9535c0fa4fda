// pk_half.hpp -- complex arithmetic on packed fp16 pairs (low half real, high half
// imaginary) with the packed-half ALU instructions.
//
// Written as vector operations, which the compiler turns into v_pk_add / mul / fma_f16 with
// the swaps and conjugations in their operand modifiers, at no instruction of their own.
// No inline assembly: the compiler does not look inside it for the wait states that gfx950
// needs between a scalar register written by the vector ALU (v_readlane) and its read as an
// operand, between a vector ALU result and the matrix product that reads it, and between a
// matrix product and the reuse of its accumulator's registers.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>

namespace rubiconv {

__device__ __forceinline__ uint32_t h2_bits(float re, float im) {  // round to nearest even
    return __builtin_bit_cast(uint32_t, __float22half2_rn(make_float2(re, im)));
}

// bf16 of f rounded to nearest even, in the low 16 bits (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

// (bf16(lo), bf16(hi)) rounded to nearest even: one v_cvt_pk_bf16_f32.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf2_bits(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ half2_t as_h2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ uint32_t h2_word(half2_t v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ half2_t lo2(half2_t a) { return half2_t{a.x, a.x}; }
__device__ __forceinline__ half2_t hi2(half2_t a) { return half2_t{a.y, a.y}; }
__device__ __forceinline__ half2_t conj2(half2_t a) { return half2_t{a.x, -a.y}; }
__device__ __forceinline__ half2_t mul_i2(half2_t a) { return half2_t{-a.y, a.x}; }      // i a
__device__ __forceinline__ half2_t fma2(half2_t a, half2_t b, half2_t c) { return __builtin_elementwise_fma(a, b, c); }

// a * b
__device__ __forceinline__ uint32_t cmul_h2(uint32_t a, uint32_t b) {
    const half2_t x = as_h2(a), y = as_h2(b);
    return h2_word(fma2(hi2(x), mul_i2(y), lo2(x) * y));
}

}  // namespace rubiconv
