// Internal: what the small-tile 16-bit kernels (igemm_mid.hip, wgrad_mid.hip) share.
#pragma once
#include <hip/hip_runtime.h>

#include "igemm_common.h"

namespace capscaps {
namespace {

constexpr unsigned OOB = 0x80000000u;           // an offset no tensor reaches: reads as zero
constexpr size_t MAX_TENSOR_BYTES = 0x70000000;  // 32-bit offsets below that mark

struct FastDiv {  // n / d for n < 2^31: (n * mul) >> shift
    unsigned mul;
    int shift;
};
inline FastDiv fast_div(unsigned d)
{
    int l = 0;
    while ((1ull << l) < d) ++l;
    return {(unsigned)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
__device__ __forceinline__ unsigned div_by(unsigned n, const FastDiv& f)
{
    return (unsigned)(((unsigned long long)n * f.mul) >> f.shift);
}

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }
inline bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
inline int log2_of(int v)
{
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4v;

// 8 K values of one column from 4 lines at LDS byte `at` and 4 at `at2` (addresses by lane as
// ds_read_b64_tr_b16 takes them)
__device__ __forceinline__ chunk_t read_transposed(char* lds, int at, int at2)
{
    struct { short4v lo, hi; } v;
    v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(lds + at));
    v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(lds + at2));
    return __builtin_bit_cast(chunk_t, v);
}
// Lane's byte offset, in a unit of 64 columns x 8 lines as the copies lay it down, of the first four
// lines of the 32 columns from `cb` on.  WIDE: 16-byte slots of 8 columns, [chunk][line], the line
// XORed with 4 in every other pair of chunks (the other four lines: address bit 6 flipped); else
// slots of 2 lines x 4 columns, [two channels or pixels][4 columns][line pair] (the others: + 512).
template <bool WIDE>
__device__ __forceinline__ int transposed_at(int lane, int cb)
{
    const int a = (lane & 15) >> 2, b = lane & 3, g = (lane >> 4) & 1;
    return WIDE ? ((cb / 8 + 2 * g + (b >> 1)) * 8 + a + 4 * g) * 16 + (b & 1) * 8
                : (cb / 4 + 4 * g + b) * 32 + a * 8;
}

}  // namespace
}  // namespace capscaps
