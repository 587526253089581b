// Internal: fp32 values as the sum of three bf16 values, 2^23 x = x1 + x2 + x3, each the rounding
// of what the ones before leave over, for the kernels that contract fp32 operands on the bf16 matrix
// instructions (Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", 2019).  3 x 8 significant bits and the signs of the remainders hold fp32's 24; the factor
// makes that hold for every magnitude: fp32's smallest step, 2^-149, becomes 2^-126, bf16's smallest
// normal value, so no term of any value, subnormal ones included, is cut off at the bottom of
// bf16's range.  (Unscaled, x3 of a value below 2^-110 would be, an absolute loss that the other
// operand multiplies: 1e-38 times 1e20 came out 3e-3 off.)  At the top, values of 2^104 and more
// and sums of 2^82 and more leave the range: they make the sum infinite or NaN (see SplitCheck).
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
// x minus one of the two values of `pair`, exact here.  Two forms: v_dot2_f32_bf16 with a pair of factors 0 and -1 is one
// instruction, but shares the matrix cores' pipe, whichever wave of the SIMD it comes from: with two waves per SIMD a
// 32x32x16 matrix instruction with two of them behind it takes 54 cycles, with four 63; alone 33, with six
// multiplications 36, six conversions 39.  Unpacking and subtracting are two instructions that run beside it.  Where
// two waves of a SIMD hide each other's issue the latter is faster (igemm32_split.hip: 543 -> 522 us), where one
// wave's issue is the limit, the former (wgrad32.hip: 672 against 680 us).  (The multiplication by SPLIT_SCALE before
// them is exact below 2^104, so contracting it with the subtraction changes no bit; above, the sums are taken again.)
__device__ __forceinline__ float minus_low(float x, unsigned pair) { return x - low_half(pair); }
__device__ __forceinline__ float minus_high(float x, unsigned pair) { return x - high_half(pair); }
// The operands of minus_bf16 for the lower and the upper value of a pair, opaque to the compiler
// (a packed inline constant would be the same value in both halves).
struct MinusOne {
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    __device__ __forceinline__ MinusOne() { asm volatile("" : "+s"(lo), "+s"(hi)); }
};
__device__ __forceinline__ float minus_bf16(float x, unsigned pair, unsigned minus_one)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, pair),
                                           __builtin_bit_cast(bf16x2v, minus_one), x, false);
}

constexpr float SPLIT_SCALE = 0x1p23f;     // of each operand
constexpr float SPLIT_UNSCALE = 0x1p-46f;  // ... and of the sums of their products, back

// Sums over split values that have to be taken again on the fp32 instructions: those that are not
// finite (an infinity, a NaN, a value or a sum that the scale factors take out of range).  A workgroup
// takes all of its sums again, one stage at a time, which is the one case where the time of a call
// depends on its data: 32 -> 32 channels of 3x3x3 capsules, N = 64, 32x32, with a NaN in every tile 1.43
// instead of 0.54 ms forward, 1.67 instead of 0.68 ms kernel gradient; one infinity in the input reaches a
// few tiles (forward 0.53 ms) but a whole range of every tap's pixels (kernel gradient 0.85 ms).
// Values of 1e-37: no difference.
struct SplitCheck {
    float poison = 0.f;
    __device__ __forceinline__ void take(const float16v& acc)
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) poison = fmaf(acc[r], 0.f, poison);  // NaN from an infinity or a NaN
    }
    __device__ __forceinline__ bool failed() const { return poison != 0.f; }
};

// The steps of splitting a pair of values: both scaled, then three times rounded, with the
// remainders taken in between.
constexpr int SPLIT_STEPS = 9;

// A kernel value the scale factor takes out of bf16's range (2^104 and more, an infinity, a NaN) is
// packed as a NaN, which spoils every sum it enters, and its 32 bits in the other two terms'
// places, for the sums taken again.
constexpr unsigned short SPLIT_MARK = 0x7fffu;
__device__ __forceinline__ void split_kernel_value(float x, unsigned short (&t)[3])
{
    const float xs = x * SPLIT_SCALE;
    t[0] = round_to_16(xs, 1);
    if ((t[0] & 0x7f80u) == 0x7f80u) {
        const unsigned bits = __builtin_bit_cast(unsigned, x);
        t[0] = SPLIT_MARK;
        t[1] = (unsigned short)(bits >> 16);
        t[2] = (unsigned short)bits;
        return;
    }
    const float r1 = xs - low_half(t[0]);
    t[1] = round_to_16(r1, 1);
    t[2] = round_to_16(r1 - low_half(t[1]), 1);
}
__device__ __forceinline__ float joined_kernel_value(unsigned t0, unsigned t1, unsigned t2)
{
    const float sum = (low_half(t0) + low_half(t1)) + low_half(t2);
    return t0 == SPLIT_MARK ? __builtin_bit_cast(float, t1 << 16 | t2) : sum * (1.f / SPLIT_SCALE);
}

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
