// Internal: fp32 values as the sum of three bf16 values, x = x1 + x2 + x3, each the rounding of
// what the ones before leave over (exact: 3 x 8 significant bits and the signs of the remainders
// hold fp32's 24), for the kernels that contract fp32 operands on the bf16 matrix instructions.
#pragma once
#include <hip/hip_runtime.h>

#include "igemm_common.h"

namespace capscaps {

// two fp32 values rounded to bf16 (the lower value in the lower half of the word)
typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned round_pair(float lo, float hi)
{
    const float2v v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2v));
}
__device__ __forceinline__ float low_half(unsigned w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float high_half(unsigned w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
// The operands of minus_bf16 for the lower and the upper value of a pair, opaque to the compiler
// (a packed inline constant would be the same value in both halves).
struct MinusOne {
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    __device__ __forceinline__ MinusOne() { asm volatile("" : "+s"(lo), "+s"(hi)); }
};
// one of the two values of `pair` times -1, plus x: exact here, and one instruction where
// unpacking the value and subtracting it are two
__device__ __forceinline__ float minus_bf16(float x, unsigned pair, unsigned minus_one)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, pair),
                                           __builtin_bit_cast(bf16x2v, minus_one), x, false);
}

// Sums over split values that have to be taken again on the fp32 instructions: those that are not
// finite (an infinity, a NaN, a value that rounds to infinity in bf16), and those that are not
// zero but below 2^-80, where operands below 2^-110, whose x3 is cut off by bf16's exponent range,
// may matter.
struct SplitCheck {
    float poison = 0.f;
    unsigned small = 0xffffffffu;
    __device__ __forceinline__ void take(const float16v& acc)
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            poison = fmaf(acc[r], 0.f, poison);  // NaN from an infinity or a NaN
            const unsigned m = 2 * __builtin_bit_cast(unsigned, acc[r]) - 1;  // zero: the largest
            small = m < small ? m : small;
        }
    }
    __device__ __forceinline__ bool failed() const { return poison != 0.f || small < ((127u - 80u) << 24); }
};

// Side operations dealt out over the gaps after matrix instructions: operation t of `count` goes into
// gap first + t * (gaps - first) / count; those of gap i are [dealt_before(i), dealt_before(i + 1)).
constexpr int dealt_before(int i, int count, int gaps, int first)
{
    int t = 0;
    while (t < count && (gaps > 1 ? first + t * (gaps - first) / count : 0) < i) ++t;
    return t;
}

// (kernel or column term, input or row term) of the six products, smallest first
constexpr int SPLIT_PRODUCTS = 6;
constexpr int SPLIT_TERM_A[SPLIT_PRODUCTS] = {2, 1, 0, 1, 0, 0};
constexpr int SPLIT_TERM_B[SPLIT_PRODUCTS] = {0, 1, 2, 0, 1, 0};

}  // namespace capscaps
