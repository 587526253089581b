// Internal: geometry of one capsule-convolution call and the launchers of the compute paths.
// Notation follows the paper's Algorithm 2 (I, K, O; taps (p,q); channels c -> m) with the
// capsule indices d0 (batch), d1 (row), d2 (contracted), d3 (column).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace capscaps {

// Raises a kernel's dynamic-LDS limit to `bytes` the first time the kernel is launched on a
// device (the attribute stays set for the process), not on every launch: the call costs host
// time on exactly the launch-bound problems.  `done` is the caller's record for that kernel, one
// bit per device.
inline hipError_t set_dynamic_lds_once(const void* kern, int bytes,
                                       std::atomic<unsigned long long>& done)
{
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    const unsigned long long bit = 1ull << (dev & 63);
    if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (err == hipSuccess && dev < 64) done.fetch_or(bit, std::memory_order_release);
    return err;
}

struct ConvShape {
    int N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3;
    int Ho, Wo;  // output extents
    int dtype;   // CAPSCAPS_FP32 / BF16 / FP16
    // output element type: 0 = fp32 (the accumulator as it is); CAPSCAPS_BF16 / FP16 = the
    // accumulator rounded to nearest even at the store (forward pass of 16-bit operands only)
    int out16 = 0;
    // Geometry overrides understood by the two tuned kernels only (launch_mfma with
    // MfmaKernel::Tuned16 or ::Dma32; everything else must be given shapes without them).  The backward
    // pass uses them to run a strided layer's input gradient as stride*stride convolutions
    // whose outputs interleave.  pad_w_set: the columns' padding is pad_w instead of pad; both
    // may then be negative (the window starts inside the image) and Ho, Wo are taken as given.
    // out_view: output pixel (n, x, y) is written at element out_base + n*out_sn + x*out_sx +
    // y*out_sy of `out` instead of densely.
    bool pad_w_set = false;
    int pad_w = 0;
    bool out_view = false;
    long long out_base = 0, out_sn = 0, out_sx = 0, out_sy = 0;
    long long out_alloc = 0;  // with out_view: elements of the whole tensor `out` points into
    // kernel_view (matrix-core paths only, honoured where the kernel tensor is repacked): kernel
    // element (p, q, c, m, d0, d2, d3) is read at element k_base + p*k_sp + q*k_sq + c*k_sc +
    // m*k_sm + d0*k_sd0 + d2*k_sd2 + d3*k_sd3 of `kernel` instead of densely (strides may be
    // negative: a flipped window).
    bool kernel_view = false;
    // in_gradient: an input gradient run as this convolution, whose kernel tensor lies transposed in
    // memory (for the choice of the kernel; set also where kernel_view is not, so that the scratch
    // asked for is that of the kernel that runs)
    bool in_gradient = false;
    // in_paired (lane-per-row kernel, 16-bit capsule rows of 4 elements): `input` already is the
    // channel-paired copy [pixel][c/2][d0][d1][c%2][d2] (a caller that runs several convolutions
    // on one input pairs it once)
    bool in_paired = false;
    long long k_base = 0, k_sp = 0, k_sq = 0, k_sc = 0, k_sm = 0, k_sd0 = 0, k_sd2 = 0, k_sd3 = 0;
    // Of this call, the small-tile kernels (mid_tiles.h): 0 = by the library's rules.  For tests: 1 = none; 2 = wherever
    // they can run, with tile `mid_tile` (negative: the estimate's) and `mid_split` pieces of the K loop (0: the
    // estimate's) as far as the workspace holds their sums.
    int mid_use = 0, mid_tile = -1, mid_split = 0;
    int padw() const { return pad_w_set ? pad_w : pad; }
    bool plain() const { return !pad_w_set && !out_view && !kernel_view && !in_paired; }
    long long pixels() const { return (long long)N * Ho * Wo; }
    size_t in_elems() const { return (size_t)N * H * W * C * D0 * D1 * D2; }
    size_t kernel_elems() const { return (size_t)kh * kw * C * M * D0 * D2 * D3; }
    size_t out_elems() const { return (size_t)N * Ho * Wo * M * D0 * D1 * D3; }
};

// Wavefront-level small-matrix path: plain FMAs, any shape, any dtype.  No scratch.
// (`out` points to fp32 or, with s.out16, to 16-bit elements; likewise for launch_mfma)
// launch_direct takes the LDS-staged wave kernel (wave_conv.hip) where it can stage the shape,
// else a thread-per-element kernel.
hipError_t launch_direct(const ConvShape& s, const void* in, const void* kernel, float* out,
                         hipStream_t stream);
bool wave_conv_eligible(const ConvShape& s);
// layers the wavefront-level path runs faster than the any-shape and the small-problem kernel, once
// they are large enough for throughput to count
inline bool few_columns(const ConvShape& s)
{
    return (long long)s.M * s.D3 <= 8 && (s.D2 % 4 != 0 || s.D3 % 4 != 0);
}
hipError_t launch_wave_conv(const ConvShape& s, const void* in, const void* kernel, float* out,
                            hipStream_t stream);

// Matrix-core path (LDS-staged implicit GEMM).  `mfma_supported` tells whether the path can
// run the shape; `mfma_workspace_bytes` is the scratch it needs (repacked kernel plus, for
// small problems, split-reduction partial sums).
// Rechunk: fp32 layers whose rows are written out in runs of four K values first (igemm_conv.hip).
enum class MfmaKernel { Auto, Generic, Tuned16, Dma32, Small, Rechunk };
// Several 16-bit convolutions whose kernels are views of one tensor (equal but for the window and k_base), on the
// tuned kernels: one repack launch for all, then each by itself.  RepackLayout: the bytes of one's repacked kernel and
// its order; 0 bytes = it needs more scratch than that, or is not for this.
constexpr int MAX_REPACK_VIEWS = 16;
struct RepackLayout {
    size_t bytes;
    int KQP, colsp, kgroup;
};
RepackLayout mfma_repack_layout(const ConvShape& s, MfmaKernel which);
hipError_t launch_repack_views(const ConvShape* f, const RepackLayout* layout, void* const* kp, int n,
                               const void* kernel, hipStream_t stream);
hipError_t launch_mfma_repacked(const ConvShape& s, const void* in, void* kp, float* out, hipStream_t stream,
                                MfmaKernel which);
bool mfma_supported(const ConvShape& s);
MfmaKernel mfma_auto_kernel(const ConvShape& s);  // what Auto resolves to (never Auto)
bool mfma_tuned16_supported(const ConvShape& s);
bool mfma_dma32_supported(const ConvShape& s);
bool mfma_small_supported(const ConvShape& s);
size_t mfma_workspace_bytes(const ConvShape& s);  // enough for every MfmaKernel choice (with
                                                  // s.out16: for Auto, the only choice then)
size_t mfma_kernel_workspace_bytes(const ConvShape& s, MfmaKernel which);  // for that kernel only
// fp32 layers on the lane-per-row kernel: what their packed kernel takes beyond its fp32 values
size_t mfma_split_overhead_bytes(const ConvShape& s);
bool igemm32_dma_fills_chip(const ConvShape& s);  // with four-wave tiles and an unsplit K loop
hipError_t launch_mfma(const ConvShape& s, const void* in, const void* kernel, float* out,
                       void* workspace, hipStream_t stream, MfmaKernel which = MfmaKernel::Auto);

// The forward pass with the library's own path choice, and the scratch it needs (defined next
// to the C ABI); used by the backward pass, which for stride 1 is two forward convolutions.  A call
// chooses once (the kernels' plans take host time that a launch-bound layer waits for).
// forward_run returns a status code of the C ABI; `status_from_hip` maps a HIP error to one and
// records it for the ABI's diagnostic call.
struct ForwardChoice {
    int path;           // CAPSCAPS_PATH_*
    MfmaKernel kernel;  // on the matrix cores
    // whether that is a matrix-core kernel, which takes the kernel tensor in place or through a repack
    // pass and therefore accepts s.kernel_view (the wavefront-level path reads it densely)
    bool takes_kernel_view;
};
ForwardChoice forward_choice(const ConvShape& s);
size_t forward_choice_bytes(const ConvShape& s, const ForwardChoice& c);
int forward_run(const ConvShape& s, const ForwardChoice& c, const void* in, const void* kernel, float* out,
                void* workspace, size_t workspace_bytes, hipStream_t stream);
// the tuned 16-bit kernel, geometry overrides allowed (EUNSUPPORTED if it cannot run the shape)
int forward_tuned16(const ConvShape& s, const void* in, const void* kernel, float* out,
                    void* workspace, size_t workspace_bytes, hipStream_t stream);
// ... and the tuned fp32 kernel
int forward_tuned32(const ConvShape& s, const void* in, const void* kernel, float* out,
                    void* workspace, size_t workspace_bytes, hipStream_t stream);
int status_from_hip(hipError_t err);

// Backward pass (backward.hip): gradients with respect to input and kernel, fp32 results.  A plan is made
// once per call; `bytes` is the scratch.
struct BwdInputPlan {
    enum Form { FullyConnected, Phases, Convolution, Gather } form;  // see backward.hip
    ForwardChoice fwd;                                               // of the first and the third
    size_t bytes;
};
BwdInputPlan bwd_input_plan(const ConvShape& s);
// which kernels run a call (for tests): tile of the small-tile kernel or -1, its pieces of the K loop, and
// else the plan's form, or for the kernel gradient 16 / 32 for wgrad16.hip / wgrad32.hip, 1 as a convolution
struct RouteInfo {
    int tile, nsplit, form;
};
RouteInfo bwd_input_route(const ConvShape& s, const BwdInputPlan& plan, size_t workspace_bytes);
RouteInfo bwd_kernel_route(const ConvShape& s, size_t need, size_t workspace_bytes);
bool bwd_input_repacks_together(const ConvShape& s, const BwdInputPlan& plan);  // (for tests) its phases' kernels
size_t bwd_kernel_workspace_bytes(const ConvShape& s);
// Return a status code of the C ABI; the caller has checked the scratch (`need`: of the kernel gradient).
int launch_bwd_input(const ConvShape& s, const BwdInputPlan& plan, const void* dout, const void* kernel,
                     float* din, void* workspace, size_t workspace_bytes, hipStream_t stream);
int launch_bwd_kernel(const ConvShape& s, size_t need, const void* input, const void* dout, float* dkernel,
                      void* workspace, size_t workspace_bytes, hipStream_t stream);

// The paper's second scheme (Algorithm 5) as a comparison implementation (scheme2.hip).
bool scheme2_supported(const ConvShape& s);
size_t scheme2_products(const ConvShape& s);  // small matrix products = index triples
hipError_t launch_scheme2_index(const ConvShape& s, int* index, hipStream_t stream);
hipError_t launch_scheme2(const ConvShape& s, const void* in, const void* kernel, float* out,
                          const int* index, hipStream_t stream);

// Measurement aid (yardstick.hip): back-to-back matrix instructions on register operands.
double yardstick_flops(int dtype, int blocks, int iters);
hipError_t launch_yardstick(int dtype, const void* seed, float* sink, int blocks, int iters,
                            hipStream_t stream);

}  // namespace capscaps
