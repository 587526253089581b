// C ABI of the capsule convolution (forward and backward pass): argument checking, path choice, launches.
// Declarations and their contracts are in include/capscaps.h.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/capscaps.h"
#include "igemm_common.h"
#include "mid_tiles.h"

using capscaps::ConvShape;
using Choice = capscaps::ForwardChoice;

namespace {

thread_local hipError_t g_last_hip_error = hipSuccess;

int hip_status(hipError_t err)
{
    if (err == hipSuccess) return CAPSCAPS_OK;
    g_last_hip_error = err;
    (void)hipGetLastError();  // leave no sticky error behind for the caller's next HIP call
    return CAPSCAPS_EHIP;
}

int fill_shape(ConvShape& s, int N, int H, int W, int C, int M, int kh, int kw, int stride, int pad,
               int D0, int D1, int D2, int D3, int dtype)
{
    if (N <= 0 || C <= 0 || M <= 0 || D0 <= 0 || D1 <= 0 || D2 <= 0 || D3 <= 0)
        return CAPSCAPS_EINVAL;
    if (dtype != CAPSCAPS_FP32 && dtype != CAPSCAPS_BF16 && dtype != CAPSCAPS_FP16)
        return CAPSCAPS_EINVAL;
    int Ho = 0, Wo = 0;
    const int rc = capscaps_out_shape(H, W, kh, kw, stride, pad, &Ho, &Wo);
    if (rc != CAPSCAPS_OK) return rc;
    // window taps are counted in 32 bits throughout (a window over a whole large scalar image,
    // 46341 x 46341 and up, would wrap)
    if ((long long)kh * kw > (1LL << 24)) return CAPSCAPS_EUNSUPPORTED;
    s = ConvShape{N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, Ho, Wo, dtype};
    // element counts must stay well inside 63 bits
    const long double big = (long double)N * H * W * C * D0 * D1 * D2;
    const long double bigo = (long double)N * Ho * Wo * M * D0 * D1 * D3;
    const long double bigk = (long double)kh * kw * C * M * D0 * D2 * D3;
    if (big > 1e17L || bigo > 1e17L || bigk > 1e17L) return CAPSCAPS_EINVAL;
    return CAPSCAPS_OK;
}

// Measured on MI355X (fp32 and bf16 layers with 3 .. 32 output columns (m, d3) and K from 4 to
// 288, the worked example of Fig. 2 among them): with 16-column tiles the matrix cores win even
// at 4 columns (12 of 16 columns of every tile are padding there, and they still finish first:
// the wavefront-level path spends more instructions staging an input value in LDS than
// multiplying it when few output columns use it).  The wavefront-level path wins
//   * where the contraction is so short (K up to 16 measured: a 1x1 or 2x2 window over one
//     channel of 4-element capsule rows) that a matrix-core tile's 64-value K slab is mostly
//     padding, and
//   * on layers of at most 8 output columns whose capsule rows are not multiples of 4 elements
//     (Fig. 2's 3x3x3 capsules: the matrix-core kernel then gathers element by element), once
//     the layer is large enough for throughput to count (a tiny one is latency-bound, and the
//     single-stage matrix-core kernel has the shorter latency);
// it also serves what the matrix-core path cannot address.
//
// The path and, on the matrix cores, the kernel.  16-bit layers below the tuned kernels' sizes and fp32 input
// gradients may run on the small-tile kernel instead (run_choice): path, scratch and what is refused for lack of
// it stay those of `kernel`, and the partial sums fit in that scratch.
Choice choose(const ConvShape& s)
{
    const Choice direct = {CAPSCAPS_PATH_DIRECT, capscaps::MfmaKernel::Auto, false};
    if (!capscaps::mfma_supported(s)) return direct;
    const long long kdim = (long long)s.kh * s.kw * s.C * s.D2;
    if (kdim <= 24) return direct;
    const double flops = 2.0 * (double)s.out_elems() * (double)kdim;
    const capscaps::MfmaKernel kernel = capscaps::mfma_auto_kernel(s);
    // (fp32 layers from 5e8 FLOPs on: the lane-per-row kernel where it is the choice, which contracts on
    // the bf16 matrix instructions -- 6x5 . 5x4 capsules, 8 columns, 9.9 GFLOP 399 against 1473 us;
    // 3x3x3 capsules, 6 columns, 0.5 GFLOP 32 against 153 us)
    const bool split32 = s.dtype == CAPSCAPS_FP32 && flops >= 5e8 &&
                         (kernel == capscaps::MfmaKernel::Dma32 || kernel == capscaps::MfmaKernel::Rechunk);
    if (!split32 && few_columns(s) && flops >= 5e7 && capscaps::wave_conv_eligible(s)) return direct;
    switch (kernel) {
        case capscaps::MfmaKernel::Tuned16: return {CAPSCAPS_PATH_MFMA_TUNED16, kernel, true};
        case capscaps::MfmaKernel::Dma32: return {CAPSCAPS_PATH_MFMA_TUNED32, kernel, true};
        case capscaps::MfmaKernel::Small: return {CAPSCAPS_PATH_MFMA_SMALL, kernel, true};
        // (the lane-per-row kernel again, but on a copy of the input that only the library's choice makes)
        case capscaps::MfmaKernel::Rechunk: return {CAPSCAPS_PATH_MFMA, kernel, true};
        default: return {CAPSCAPS_PATH_MFMA_GENERIC, kernel, true};
    }
}
size_t scratch_bytes(const ConvShape& s, const Choice& c)
{
    return c.path == CAPSCAPS_PATH_DIRECT ? 0 : capscaps::mfma_kernel_workspace_bytes(s, c.kernel);
}

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Scratch of the entry point that allocates nothing (capscaps_conv_fwd_static): a fixed array in
// every GPU's memory, there from the moment the library's code is loaded on that GPU until the
// process ends.  In host code the array's name stands for the symbol, not for a device address:
// the address on the current device is looked up once per device and kept.  The array is larger
// than the limit callers are told: an fp32 kernel tensor is packed as three bf16 terms, half as
// much again as fp32 values (and rounded up to whole tiles), and the limit counts the values.
constexpr size_t SCRATCH_LIMIT = CAPSCAPS_STATIC_SCRATCH_BYTES;
constexpr size_t SCRATCH_ARRAY = (size_t)128 << 20;
static __device__ __align__(256) unsigned char scratch[SCRATCH_ARRAY];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** ptr)
{
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return hip_status(err);
    if (dev < 0 || dev >= kMaxDevices) return CAPSCAPS_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return hip_status(err);
        if (p == nullptr) return CAPSCAPS_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return CAPSCAPS_OK;
}

bool fits_scratch(const ConvShape& s, const Choice& own)
{
    const size_t need = scratch_bytes(s, own);
    if (need <= SCRATCH_LIMIT) return true;
    return need <= SCRATCH_ARRAY && s.dtype == CAPSCAPS_FP32 && own.path == CAPSCAPS_PATH_MFMA_TUNED32 &&
           need - capscaps::mfma_split_overhead_bytes(s) <= SCRATCH_LIMIT;
}

// A kernel whose scratch fits where that of the library's own choice does not; Auto: none.  The
// lane-per-row kernel is the choice that may need too much: for the copy of the input with its
// channels paired (16-bit capsule rows of 4), for an fp32 kernel tensor in bf16 terms, for the partial
// sums of its large tiles.  16-bit layers that fill the chip with its tiles are refused instead.
capscaps::MfmaKernel leaner_kernel(const ConvShape& s, const Choice& own)
{
    using capscaps::MfmaKernel;
    if (s.dtype != CAPSCAPS_FP32 &&
        (own.path != CAPSCAPS_PATH_MFMA_TUNED32 || capscaps::igemm32_dma_fills_chip(s)))
        return MfmaKernel::Auto;
    if (capscaps::mfma_kernel_workspace_bytes(s, MfmaKernel::Generic) <= SCRATCH_LIMIT)
        return MfmaKernel::Generic;
    if (s.dtype == CAPSCAPS_FP32 && capscaps::mfma_small_supported(s) &&
        capscaps::mfma_kernel_workspace_bytes(s, MfmaKernel::Small) <= SCRATCH_LIMIT)
        return MfmaKernel::Small;
    return MfmaKernel::Auto;
}

capscaps::MidPick small_tiles(const ConvShape& s, const Choice& c, size_t need, size_t workspace_bytes)
{
    if (c.path == CAPSCAPS_PATH_DIRECT && s.mid_use != 2) return {};
    return capscaps::igemm_mid_choice(s, c.kernel, s.mid_use == 2 ? workspace_bytes : need);
}

// The library's own choice; it needs scratch for the kernel it picks only.
int run_choice(const void* input, const void* kernel, void* out, const ConvShape& s, const Choice& c,
               void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    float* dst = static_cast<float*>(out);
    const size_t need = scratch_bytes(s, c);
    if (need > 0 && (workspace == nullptr || workspace_bytes < need)) return CAPSCAPS_EWORKSPACE;
    if (need > 0 && misaligned(workspace)) return CAPSCAPS_EINVAL;
    if (const capscaps::MidPick pick = small_tiles(s, c, need, workspace_bytes))
        return hip_status(
            capscaps::launch_igemm_mid(&s, 1, s.kernel_elems(), pick, input, kernel, dst, workspace, stream));
    if (c.path == CAPSCAPS_PATH_DIRECT)
        return hip_status(capscaps::launch_direct(s, input, kernel, dst, stream));
    return hip_status(capscaps::launch_mfma(s, input, kernel, dst, workspace, stream, c.kernel));
}

int run(const void* input, const void* kernel, void* out, const ConvShape& s, int path,
        void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    hipError_t err;
    if (path == CAPSCAPS_PATH_AUTO) {
        return run_choice(input, kernel, out, s, choose(s), workspace, workspace_bytes, stream);
    } else if (path == CAPSCAPS_PATH_DIRECT) {
        err = capscaps::launch_direct(s, input, kernel, static_cast<float*>(out), stream);
    } else if (path == CAPSCAPS_PATH_MFMA || path == CAPSCAPS_PATH_MFMA_GENERIC ||
               path == CAPSCAPS_PATH_MFMA_TUNED16 || path == CAPSCAPS_PATH_MFMA_TUNED32 ||
               path == CAPSCAPS_PATH_MFMA_SMALL) {
        if (!capscaps::mfma_supported(s)) return CAPSCAPS_EUNSUPPORTED;
        if (path == CAPSCAPS_PATH_MFMA)
            return run_choice(input, kernel, out, s, {path, capscaps::mfma_auto_kernel(s), true}, workspace,
                              workspace_bytes, stream);
        if (path == CAPSCAPS_PATH_MFMA_TUNED16 && !capscaps::mfma_tuned16_supported(s))
            return CAPSCAPS_EUNSUPPORTED;
        if (path == CAPSCAPS_PATH_MFMA_TUNED32 && !capscaps::mfma_dma32_supported(s))
            return CAPSCAPS_EUNSUPPORTED;
        if (path == CAPSCAPS_PATH_MFMA_SMALL && !capscaps::mfma_small_supported(s))
            return CAPSCAPS_EUNSUPPORTED;
        const capscaps::MfmaKernel which =
            path == CAPSCAPS_PATH_MFMA_GENERIC   ? capscaps::MfmaKernel::Generic
            : path == CAPSCAPS_PATH_MFMA_TUNED16 ? capscaps::MfmaKernel::Tuned16
            : path == CAPSCAPS_PATH_MFMA_SMALL   ? capscaps::MfmaKernel::Small
                                                 : capscaps::MfmaKernel::Dma32;
        // a forced kernel is held to the size that covers every one (what the size query reports)
        const size_t need = capscaps::mfma_workspace_bytes(s);
        if (need > 0 && (workspace == nullptr || workspace_bytes < need))
            return CAPSCAPS_EWORKSPACE;
        if (need > 0 && misaligned(workspace)) return CAPSCAPS_EINVAL;
        err = capscaps::launch_mfma(s, input, kernel, static_cast<float*>(out), workspace, stream,
                                    which);
    } else {
        return CAPSCAPS_EINVAL;
    }
    return hip_status(err);
}

}  // namespace

namespace capscaps {

int status_from_hip(hipError_t err) { return hip_status(err); }

ForwardChoice forward_choice(const ConvShape& s) { return choose(s); }

size_t forward_choice_bytes(const ConvShape& s, const ForwardChoice& c) { return scratch_bytes(s, c); }

int forward_run(const ConvShape& s, const ForwardChoice& c, const void* in, const void* kernel, float* out,
                void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (s.pad_w_set || s.out_view) return CAPSCAPS_EINVAL;
    if (s.kernel_view && !c.takes_kernel_view) return CAPSCAPS_EINVAL;
    return run_choice(in, kernel, out, s, c, workspace, workspace_bytes, stream);
}

MidPick forward_small_tiles(const ConvShape& s, const ForwardChoice& c, size_t workspace_bytes)
{
    return small_tiles(s, c, scratch_bytes(s, c), workspace_bytes);
}

int forward_tuned16(const ConvShape& s, const void* in, const void* kernel, float* out,
                    void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    return run(in, kernel, out, s, CAPSCAPS_PATH_MFMA_TUNED16, workspace, workspace_bytes, stream);
}

int forward_tuned32(const ConvShape& s, const void* in, const void* kernel, float* out,
                    void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    return run(in, kernel, out, s, CAPSCAPS_PATH_MFMA_TUNED32, workspace, workspace_bytes, stream);
}

}  // namespace capscaps

extern "C" {

int capscaps_out_shape(int H, int W, int kh, int kw, int stride, int pad, int* Ho, int* Wo)
{
    if (Ho == nullptr || Wo == nullptr) return CAPSCAPS_EINVAL;
    if (H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || stride <= 0 || pad < 0) return CAPSCAPS_EINVAL;
    if (pad > (1 << 28) || H > (1 << 28) || W > (1 << 28)) return CAPSCAPS_EINVAL;
    if (kh > H + 2 * pad || kw > W + 2 * pad) return CAPSCAPS_EINVAL;
    *Ho = (H + 2 * pad - kh) / stride + 1;
    *Wo = (W + 2 * pad - kw) / stride + 1;
    return CAPSCAPS_OK;
}

size_t capscaps_conv_fwd_workspace_bytes(int N, int H, int W, int C, int M, int kh, int kw,
                                         int stride, int pad, int D0, int D1, int D2, int D3,
                                         int dtype)
{
    ConvShape s;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    return capscaps::mfma_workspace_bytes(s);
}

int capscaps_select_path(int N, int H, int W, int C, int M, int kh, int kw, int stride, int pad,
                         int D0, int D1, int D2, int D3, int dtype)
{
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    return choose(s).path;
}

int capscaps_conv_fwd_path(const void* input, const void* kernel, void* out, int N, int H, int W,
                           int C, int M, int kh, int kw, int stride, int pad, int D0, int D1,
                           int D2, int D3, int dtype, int path, void* workspace,
                           size_t workspace_bytes, void* stream)
{
    if (input == nullptr || kernel == nullptr || out == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(kernel) || misaligned(out)) return CAPSCAPS_EINVAL;
    if (path < CAPSCAPS_PATH_AUTO || path > CAPSCAPS_PATH_MFMA_SMALL) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    return run(input, kernel, out, s, path, workspace, workspace_bytes,
               static_cast<hipStream_t>(stream));
}

int capscaps_conv_fwd_ex(const void* input, const void* kernel, void* out, int N, int H, int W,
                         int C, int M, int kh, int kw, int stride, int pad, int D0, int D1, int D2,
                         int D3, int dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    return capscaps_conv_fwd_path(input, kernel, out, N, H, W, C, M, kh, kw, stride, pad, D0, D1,
                                  D2, D3, dtype, CAPSCAPS_PATH_AUTO, workspace, workspace_bytes,
                                  stream);
}

size_t capscaps_conv_fwd_out16_workspace_bytes(int N, int H, int W, int C, int M, int kh, int kw,
                                               int stride, int pad, int D0, int D1, int D2, int D3,
                                               int dtype)
{
    ConvShape s;
    if (dtype != CAPSCAPS_BF16 && dtype != CAPSCAPS_FP16) return 0;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    s.out16 = dtype;
    return scratch_bytes(s, choose(s));
}

int capscaps_conv_fwd_out16(const void* input, const void* kernel, void* out, int N, int H, int W,
                            int C, int M, int kh, int kw, int stride, int pad, int D0, int D1,
                            int D2, int D3, int dtype, void* workspace, size_t workspace_bytes,
                            void* stream)
{
    if (input == nullptr || kernel == nullptr || out == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(kernel) || misaligned(out)) return CAPSCAPS_EINVAL;
    if (dtype != CAPSCAPS_BF16 && dtype != CAPSCAPS_FP16) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    s.out16 = dtype;
    return run(input, kernel, out, s, CAPSCAPS_PATH_AUTO, workspace, workspace_bytes,
               static_cast<hipStream_t>(stream));
}

int capscaps_conv_fwd(const void* input, const void* kernel, void* out, int N, int H, int W, int C,
                      int M, int kh, int kw, int stride, int D0, int D1, int D2, int D3, int dtype,
                      void* stream)
{
    if (input == nullptr || kernel == nullptr || out == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(kernel) || misaligned(out)) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, 0, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Choice own = choose(s);
    const size_t need = scratch_bytes(s, own);
    void* ws = nullptr;
    if (need > 0) {
        const hipError_t err = hipMallocAsync(&ws, need, st);
        if (err != hipSuccess) return hip_status(err);
    }
    const int status = run_choice(input, kernel, out, s, own, ws, need, st);
    if (ws != nullptr) {
        const hipError_t err = hipFreeAsync(ws, st);
        if (err != hipSuccess && status == CAPSCAPS_OK) return hip_status(err);
    }
    return status;
}

int capscaps_conv_fwd_static(const void* input, const void* kernel, void* out, int N, int H, int W,
                             int C, int M, int kh, int kw, int stride, int pad, int D0, int D1,
                             int D2, int D3, int dtype, void* stream)
{
    if (input == nullptr || kernel == nullptr || out == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(kernel) || misaligned(out)) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    const Choice own = choose(s);
    capscaps::MfmaKernel lean = capscaps::MfmaKernel::Auto;
    if (!fits_scratch(s, own)) {
        lean = leaner_kernel(s, own);
        if (lean == capscaps::MfmaKernel::Auto) return CAPSCAPS_ESCRATCH;
    }
    void* ws = nullptr;
    const int rs = scratch_of_current_device(&ws);
    if (rs != CAPSCAPS_OK) return rs;
    if (lean != capscaps::MfmaKernel::Auto)
        return hip_status(capscaps::launch_mfma(s, input, kernel, static_cast<float*>(out), ws,
                                                static_cast<hipStream_t>(stream), lean));
    return run_choice(input, kernel, out, s, own, ws, SCRATCH_ARRAY, static_cast<hipStream_t>(stream));
}

size_t capscaps_conv_bwd_input_workspace_bytes(int N, int H, int W, int C, int M, int kh, int kw,
                                               int stride, int pad, int D0, int D1, int D2, int D3,
                                               int dtype)
{
    ConvShape s;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    return capscaps::bwd_input_plan(s).bytes;
}

size_t capscaps_conv_bwd_kernel_workspace_bytes(int N, int H, int W, int C, int M, int kh, int kw,
                                                int stride, int pad, int D0, int D1, int D2,
                                                int D3, int dtype)
{
    ConvShape s;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    return capscaps::bwd_kernel_workspace_bytes(s);
}

int capscaps_conv_bwd_input(const void* dout, const void* kernel, void* dinput, int N, int H, int W,
                            int C, int M, int kh, int kw, int stride, int pad, int D0, int D1,
                            int D2, int D3, int dtype, void* workspace, size_t workspace_bytes,
                            void* stream)
{
    if (dout == nullptr || kernel == nullptr || dinput == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(dout) || misaligned(kernel) || misaligned(dinput)) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    const capscaps::BwdInputPlan plan = capscaps::bwd_input_plan(s);
    if (plan.bytes > 0 && (workspace == nullptr || workspace_bytes < plan.bytes)) return CAPSCAPS_EWORKSPACE;
    if (plan.bytes > 0 && misaligned(workspace)) return CAPSCAPS_EINVAL;
    return capscaps::launch_bwd_input(s, plan, dout, kernel, static_cast<float*>(dinput), workspace,
                                      workspace_bytes, static_cast<hipStream_t>(stream));
}

size_t capscaps_conv_bwd_input_out16_workspace_bytes(int N, int H, int W, int C, int M, int kh,
                                                     int kw, int stride, int pad, int D0, int D1,
                                                     int D2, int D3, int dtype)
{
    ConvShape s;
    if (dtype != CAPSCAPS_BF16 && dtype != CAPSCAPS_FP16) return 0;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    s.out16 = dtype;
    return capscaps::bwd_input_plan(s).bytes;
}

int capscaps_conv_bwd_input_out16(const void* dout, const void* kernel, void* dinput, int N, int H,
                                  int W, int C, int M, int kh, int kw, int stride, int pad, int D0,
                                  int D1, int D2, int D3, int dtype, void* workspace,
                                  size_t workspace_bytes, void* stream)
{
    if (dout == nullptr || kernel == nullptr || dinput == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(dout) || misaligned(kernel) || misaligned(dinput)) return CAPSCAPS_EINVAL;
    if (dtype != CAPSCAPS_BF16 && dtype != CAPSCAPS_FP16) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    s.out16 = dtype;
    const capscaps::BwdInputPlan plan = capscaps::bwd_input_plan(s);
    if (plan.bytes > 0 && (workspace == nullptr || workspace_bytes < plan.bytes)) return CAPSCAPS_EWORKSPACE;
    if (plan.bytes > 0 && misaligned(workspace)) return CAPSCAPS_EINVAL;
    return capscaps::launch_bwd_input(s, plan, dout, kernel, static_cast<float*>(dinput), workspace,
                                      workspace_bytes, static_cast<hipStream_t>(stream));
}

int capscaps_conv_bwd_kernel(const void* input, const void* dout, void* dkernel, int N, int H,
                             int W, int C, int M, int kh, int kw, int stride, int pad, int D0,
                             int D1, int D2, int D3, int dtype, void* workspace,
                             size_t workspace_bytes, void* stream)
{
    if (input == nullptr || dout == nullptr || dkernel == nullptr) return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(dout) || misaligned(dkernel)) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    const size_t need = capscaps::bwd_kernel_workspace_bytes(s);
    if (need > 0 && (workspace == nullptr || workspace_bytes < need)) return CAPSCAPS_EWORKSPACE;
    if (need > 0 && misaligned(workspace)) return CAPSCAPS_EINVAL;
    return capscaps::launch_bwd_kernel(s, need, input, dout, static_cast<float*>(dkernel), workspace,
                                       workspace_bytes, static_cast<hipStream_t>(stream));
}

size_t capscaps_scheme2_index_bytes(int N, int H, int W, int C, int M, int kh, int kw, int stride,
                                    int pad, int D0, int D1, int D2, int D3, int dtype)
{
    ConvShape s;
    if (fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype) != CAPSCAPS_OK)
        return 0;
    if (!capscaps::scheme2_supported(s)) return 0;
    return capscaps::scheme2_products(s) * 3 * sizeof(int);
}

int capscaps_scheme2_build_index(void* index, size_t index_bytes, int N, int H, int W, int C, int M,
                                 int kh, int kw, int stride, int pad, int D0, int D1, int D2,
                                 int D3, int dtype, void* stream)
{
    if (index == nullptr || misaligned(index)) return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    if (!capscaps::scheme2_supported(s)) return CAPSCAPS_EUNSUPPORTED;
    if (index_bytes < capscaps::scheme2_products(s) * 3 * sizeof(int)) return CAPSCAPS_EWORKSPACE;
    return hip_status(capscaps::launch_scheme2_index(s, static_cast<int*>(index),
                                                     static_cast<hipStream_t>(stream)));
}

int capscaps_scheme2_fwd(const void* input, const void* kernel, void* out, const void* index,
                         size_t index_bytes, int N, int H, int W, int C, int M, int kh, int kw,
                         int stride, int pad, int D0, int D1, int D2, int D3, int dtype,
                         void* stream)
{
    if (input == nullptr || kernel == nullptr || out == nullptr || index == nullptr)
        return CAPSCAPS_EINVAL;
    if (misaligned(input) || misaligned(kernel) || misaligned(out) || misaligned(index))
        return CAPSCAPS_EINVAL;
    ConvShape s;
    const int rc = fill_shape(s, N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3, dtype);
    if (rc != CAPSCAPS_OK) return rc;
    if (!capscaps::scheme2_supported(s)) return CAPSCAPS_EUNSUPPORTED;
    if (index_bytes < capscaps::scheme2_products(s) * 3 * sizeof(int)) return CAPSCAPS_EWORKSPACE;
    return hip_status(capscaps::launch_scheme2(s, input, kernel, static_cast<float*>(out),
                                               static_cast<const int*>(index),
                                               static_cast<hipStream_t>(stream)));
}

double capscaps_mfma_yardstick_flops(int dtype, int blocks, int iters)
{
    if (dtype < 0 || dtype > 2 || blocks <= 0 || iters <= 0) return 0.0;
    return capscaps::yardstick_flops(dtype, blocks, iters);
}

int capscaps_mfma_yardstick(const void* seed, void* sink, int dtype, int blocks, int iters,
                            void* stream)
{
    if (seed == nullptr || sink == nullptr || misaligned(seed) || misaligned(sink))
        return CAPSCAPS_EINVAL;
    if (dtype < 0 || dtype > 2 || blocks <= 0 || blocks > (1 << 20) || iters <= 0 ||
        iters > (1 << 24))
        return CAPSCAPS_EINVAL;
    return hip_status(capscaps::launch_yardstick(dtype, seed, static_cast<float*>(sink), blocks,
                                                 iters, static_cast<hipStream_t>(stream)));
}

// For the tests and bench.py only (not in the header): a forward pass (op 0), input (1) or kernel gradient (2) with or without the
// small-tile kernels, and which kernels would run.  `shape`: N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3,
// dtype; `small_tiles`: ConvShape::mid_use, mid_tile, mid_split; `info`: RouteInfo (forward: form = the path).
namespace {
int testing_shape(ConvShape& s, const int* a, int out16, const int* small_tiles)
{
    const int rc = fill_shape(s, a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13]);
    if (rc != CAPSCAPS_OK) return rc;
    s.out16 = out16 ? s.dtype : 0;
    s.mid_use = small_tiles[0];
    s.mid_tile = small_tiles[1];
    s.mid_split = small_tiles[2];
    return CAPSCAPS_OK;
}
}  // namespace

int capscaps_testing_conv(int op, const int* shape, int out16, const int* small_tiles, const void* a, const void* b,
                          void* out, void* workspace, size_t workspace_bytes, void* stream)
{
    ConvShape s;
    const int rc = testing_shape(s, shape, out16, small_tiles);
    if (rc != CAPSCAPS_OK) return rc;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    if (op == 0) return run(a, b, out, s, CAPSCAPS_PATH_AUTO, workspace, workspace_bytes, st);
    const capscaps::BwdInputPlan plan = op == 1 ? capscaps::bwd_input_plan(s) : capscaps::BwdInputPlan{};
    const size_t need = op == 1 ? plan.bytes : capscaps::bwd_kernel_workspace_bytes(s);
    if (need > 0 && (workspace == nullptr || workspace_bytes < need)) return CAPSCAPS_EWORKSPACE;
    if (op == 1)
        return capscaps::launch_bwd_input(s, plan, a, b, static_cast<float*>(out), workspace, workspace_bytes, st);
    return capscaps::launch_bwd_kernel(s, need, a, b, static_cast<float*>(out), workspace, workspace_bytes, st);
}

int capscaps_testing_route(int op, const int* shape, int out16, const int* small_tiles, size_t workspace_bytes,
                           int* info)
{
    ConvShape s;
    const int rc = testing_shape(s, shape, out16, small_tiles);
    if (rc != CAPSCAPS_OK) return rc;
    capscaps::RouteInfo r{};
    if (op == 0) {
        const Choice c = choose(s);
        const capscaps::MidPick pick = capscaps::forward_small_tiles(s, c, workspace_bytes);
        r = {pick.tile, pick.nsplit, c.path};
    } else if (op == 1) {
        r = capscaps::bwd_input_route(s, capscaps::bwd_input_plan(s), workspace_bytes);
    } else {
        r = capscaps::bwd_kernel_route(s, capscaps::bwd_kernel_workspace_bytes(s), workspace_bytes);
    }
    info[0] = r.tile;
    info[1] = r.nsplit;
    info[2] = r.form;
    return CAPSCAPS_OK;
}

// 1: one launch repacks the kernels of this input gradient's phases; 0: there is none, or a launch for each
int capscaps_testing_repacks_together(const int* shape, int out16, const int* small_tiles)
{
    ConvShape s;
    if (testing_shape(s, shape, out16, small_tiles) != CAPSCAPS_OK) return 0;
    return capscaps::bwd_input_repacks_together(s, capscaps::bwd_input_plan(s));
}

const char* capscaps_last_hip_error(void) { return hipGetErrorString(g_last_hip_error); }

const char* capscaps_strerror(int status)
{
    switch (status) {
        case CAPSCAPS_OK: return "success";
        case CAPSCAPS_EINVAL: return "invalid argument";
        case CAPSCAPS_EWORKSPACE: return "workspace missing or too small";
        case CAPSCAPS_EUNSUPPORTED: return "path does not support this shape";
        case CAPSCAPS_EHIP: return "HIP runtime error";
        case CAPSCAPS_ESCRATCH:
            return "problem needs more scratch than the fixed buffer of the entry point that "
                   "allocates nothing";
        default: return "unknown status";
    }
}

}  // extern "C"
