// Internal: the small-tile kernels (igemm_mid.hip, wgrad_mid.hip), and what they share.
#pragma once
#include <hip/hip_runtime.h>

#include "igemm_common.h"

namespace capscaps {

// Tile (an index into the kernel's table; negative: the layer stays on another kernel) and pieces of the K loop.
struct MidPick {
    int tile = -1, nsplit = 1;
    explicit operator bool() const { return tile >= 0; }
};
struct MidEstimate {
    MidPick pick;
    double us;
};

// what a test asked for (ConvShape::mid_use = 2)
inline MidPick asked_pick(const ConvShape& s, MidPick pick, int tiles, double out_bytes, size_t room)
{
    if (s.mid_tile >= 0) pick.tile = s.mid_tile % tiles;
    const double fit = (double)room / out_bytes;
    if (s.mid_split > 0) pick.nsplit = s.mid_split <= fit ? s.mid_split : fit >= 1 ? (int)fit : 1;
    return pick;
}

// Forward pass (16-bit) and input gradient of layers below the tuned kernels' sizes (igemm_mid.hip): one launch,
// kernel tensor read in place, tiles of 64 or 128 rows and columns.  `f`: one forward pass, or an input gradient as
// one convolution or as the n phases of a strided layer (all written by the one launch; geometry
// overrides allowed).  `kernel_elems`: of the whole kernel tensor.  Partial sums of a split K loop take
// at most `room` bytes of the workspace.  `skip_taps` (input gradients): an infinite or NaN kernel value reaches
// only the pixels that its tap reaches (otherwise also, as a NaN, those whose tap lies outside the image).
bool igemm_mid_eligible(const ConvShape* f, int n, size_t kernel_elems);
MidEstimate igemm_mid_best(const ConvShape* f, int n, size_t room);  // the least estimated time
// the library's choice for a convolution that `otherwise` would run
MidPick igemm_mid_choice(const ConvShape& s, MfmaKernel otherwise, size_t room);
// ... that a forward pass with the library's choice `c` runs on (capscaps_api.hip)
MidPick forward_small_tiles(const ConvShape& s, const ForwardChoice& c, size_t workspace_bytes);
// estimated time of Tuned16 or Dma32, us
double igemm16_tuned_us(const ConvShape& s, MfmaKernel which);
// ... of the fp32 kernels (igemm32_dma.hip)
double igemm32_us(const ConvShape& s, MfmaKernel which);
hipError_t launch_igemm_mid(const ConvShape* f, int n, size_t kernel_elems, MidPick pick, const void* in,
                            const void* kernel, float* out, void* workspace, hipStream_t stream,
                            bool skip_taps = false);

// Kernel gradient of such layers (wgrad_mid.hip); partial sums take at most `room` bytes
bool wgrad_mid_eligible(const ConvShape& s);
MidPick wgrad_mid_choice(const ConvShape& s, size_t room);  // the library's
hipError_t launch_wgrad_mid(const ConvShape& s, MidPick pick, const void* input, const void* dout, float* dkernel,
                            void* workspace, hipStream_t stream);
double wgrad32_us(const ConvShape& s);  // estimated time of launch_wgrad32, us

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
