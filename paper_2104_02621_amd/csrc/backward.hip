// Backward pass of the capsule convolution: gradients with respect to the input and to the
// kernel (the two results of the paper's Algorithm 4, taken as the derivative of Algorithm 2's
// sum, since the printed algorithm is garbled).  With G = dL/dO:
//
//   dI[n,h,w,c,d0] (D1xD2) = sum_{x*s+p-pad=h, y*s+q-pad=w, m}  G[n,x,y,m,d0] (D1xD3) . K[p,q,c,m,d0]^T
//   dK[p,q,c,m,d0] (D2xD3) = sum_{n,x,y}  I[n,x*s+p-pad,y*s+q-pad,c,d0]^T (D2xD1) . G[n,x,y,m,d0] (D1xD3)
//
// dK has kernels of its own for the common capsule shapes (wgrad16.hip, wgrad32.hip: one GEMM per
// window tap over the output pixels the tap reaches); this file holds dI and the fallback for dK.
// For stride 1 both are capsule convolutions themselves and run on the forward kernels:
//   dI = conv_fwd(G, K'),  K'[kh-1-p][kw-1-q][m][c][d0][d3][d2] = K[p][q][c][m][d0][d2][d3],
//        padding kh-1-pad (square windows), channels M -> C, capsules (D1xD3).(D3xD2);
//   dK = conv_fwd(I', G'), I' = I as [C][H][W][N][D0][D2][D1] (images <-> channels, capsules
//        transposed), G' = G as [H'][W'][N][M][D0][D1][D3] (the output gradient is the window),
//        same padding; the result [C][kh][kw][M][D0][D2][D3] is permuted into the kernel layout.
// A stride s > 1 splits dI into s*s phases, the pixels with equal ((h+pad) mod s, (w+pad) mod s):
// phase (a,b) is a stride-1 convolution of G with the window taps p = a, a+s, ..., q = b, b+s, ...
// (flipped), whose output pixels lie s apart in dI.  Where every phase fits a tuned forward
// kernel (for the lane-per-row one: where it is the library's choice) that kernel runs each phase
// with its own row and column padding and writes through an output stride: no multiplication
// by zeros.  Otherwise the output gradient is spread out: G is copied into a zero
// buffer of the stride-1 output extent (H+2*pad-kh+1 rows), pixel (x,y) at (x*s, y*s).  The
// contraction then runs over s*s times the needed terms (the zeros), but on the matrix cores.
// The fully-connected layer's dI (one output pixel, window = image) is a 1x1 convolution whose
// output channels are the (h,w,c) of the input.  The layout changes are done by one strided
// copy kernel.  What these forms do not cover (dI with a non-square window or pad > kh-1)
// takes the small-tile kernel (igemm_mid.hip), or, for capsules it cannot run, a plain gather
// kernel, one thread per element of dI.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "igemm_common.h"
#include "mid_tiles.h"

namespace capscaps {
namespace {

// Strided copy over a 7-D index space: dst[dst_base + sum c_k*dst_stride_k] =
// src[src_base + sum c_k*src_stride_k] for every index c (last coordinate fastest).
struct Permute7 {
    long long dim[7];
    long long src_stride[7];
    long long src_base;
    long long dst_stride[7];
    long long dst_base;
};

// dense destination of extents dim[]: element strides of a row-major array
Permute7 gather_into_dense(const long long (&dim)[7], const long long (&src_stride)[7],
                           long long src_base)
{
    Permute7 pm{};
    long long st = 1;
    for (int k = 6; k >= 0; --k) {
        pm.dim[k] = dim[k];
        pm.src_stride[k] = src_stride[k];
        pm.dst_stride[k] = st;
        st *= dim[k];
    }
    pm.src_base = src_base;
    pm.dst_base = 0;
    return pm;
}

template <typename T>
__global__ __launch_bounds__(256) void permute7_kernel(const T* __restrict__ src,
                                                       T* __restrict__ dst, Permute7 pm,
                                                       long long total)
{
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
    if (id >= total) return;
    long long r = id, so = pm.src_base, dofs = pm.dst_base;
#pragma unroll
    for (int k = 6; k >= 0; --k) {
        const long long c = r % pm.dim[k];
        r /= pm.dim[k];
        so += c * pm.src_stride[k];
        dofs += c * pm.dst_stride[k];
    }
    dst[dofs] = src[so];
}

// bytes is a multiple of 16
__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* __restrict__ dst, size_t chunks)
{
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (id < chunks) dst[id] = make_uint4(0u, 0u, 0u, 0u);
}

hipError_t launch_fill_zero(void* dst, size_t bytes, hipStream_t stream)
{
    const size_t chunks = bytes / 16, blocks = (chunks + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    fill_zero_kernel<<<(unsigned)blocks, 256, 0, stream>>>(static_cast<uint4*>(dst), chunks);
    return hipGetLastError();
}

hipError_t launch_permute(const void* src, void* dst, const Permute7& pm, int elem_bytes,
                          hipStream_t stream)
{
    long long total = 1;
    for (int k = 0; k < 7; ++k) total *= pm.dim[k];
    const long long blocks = (total + 255) / 256;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (elem_bytes == 4)
        permute7_kernel<float><<<(unsigned)blocks, 256, 0, stream>>>((const float*)src, (float*)dst,
                                                                     pm, total);
    else
        permute7_kernel<unsigned short><<<(unsigned)blocks, 256, 0, stream>>>(
            (const unsigned short*)src, (unsigned short*)dst, pm, total);
    return hipGetLastError();
}

template <typename T>
__device__ __forceinline__ float to_f32(T v);
template <>
__device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float to_f32<__half>(__half v) { return __half2float(v); }
template <>
__device__ __forceinline__ float to_f32<__hip_bfloat16>(__hip_bfloat16 v)
{
    return __bfloat162float(v);
}

// dI, any stride, window and padding: one thread per element of dI, gather over taps, m, d3.
template <typename T>
__global__ __launch_bounds__(256) void bwd_input_direct_kernel(const T* __restrict__ G,
                                                               const T* __restrict__ K,
                                                               float* __restrict__ dI, ConvShape s,
                                                               size_t total)
{
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    size_t r = e;
    const int d2 = (int)(r % s.D2); r /= s.D2;
    const int d1 = (int)(r % s.D1); r /= s.D1;
    const int d0 = (int)(r % s.D0); r /= s.D0;
    const int c = (int)(r % s.C);   r /= s.C;
    const int w = (int)(r % s.W);   r /= s.W;
    const int h = (int)(r % s.H);   r /= s.H;
    const int n = (int)r;
    const size_t g_caps = (size_t)s.D0 * s.D1 * s.D3, k_caps = (size_t)s.D0 * s.D2 * s.D3;
    float acc = 0.f;
    for (int p = 0; p < s.kh; ++p) {
        const int hx = h + s.pad - p;
        if (hx < 0 || hx % s.stride != 0 || hx / s.stride >= s.Ho) continue;
        for (int q = 0; q < s.kw; ++q) {
            const int wy = w + s.pad - q;
            if (wy < 0 || wy % s.stride != 0 || wy / s.stride >= s.Wo) continue;
            const int x = hx / s.stride, y = wy / s.stride;
            const T* gp = G + (((size_t)n * s.Ho + x) * s.Wo + y) * s.M * g_caps +
                          ((size_t)d0 * s.D1 + d1) * s.D3;
            const T* kp = K + (((size_t)p * s.kw + q) * s.C + c) * s.M * k_caps +
                          ((size_t)d0 * s.D2 + d2) * s.D3;
            for (int m = 0; m < s.M; ++m) {
                for (int d3 = 0; d3 < s.D3; ++d3)
                    acc = fmaf(to_f32(gp[d3]), to_f32(kp[d3]), acc);
                gp += g_caps;
                kp += k_caps;
            }
        }
    }
    store1(dI, (long long)e, acc, s.out16);
}

template <typename Kern, typename... Args>
hipError_t launch_1d(Kern kern, size_t total, hipStream_t stream, Args... args)
{
    const size_t blocks = (total + 255) / 256;
    if (blocks == 0 || blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    kern<<<(unsigned)blocks, 256, 0, stream>>>(args..., total);
    return hipGetLastError();
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }
int elem_bytes(const ConvShape& s) { return s.dtype == 0 ? 4 : 2; }

void same_small_tiles(ConvShape& f, const ConvShape& s)
{
    f.mid_use = s.mid_use;
    f.mid_tile = s.mid_tile;
    f.mid_split = s.mid_split;
}

// extents of the output gradient spread out to stride 1
int spread_h(const ConvShape& s) { return s.H + 2 * s.pad - s.kh + 1; }
int spread_w(const ConvShape& s) { return s.W + 2 * s.pad - s.kw + 1; }
size_t spread_elems(const ConvShape& s)
{
    return (size_t)s.N * spread_h(s) * spread_w(s) * s.M * s.D0 * s.D1 * s.D3;
}

// One dimension of a phase of the strided input gradient: the positions h with (h + pad) mod s
// == a are h = s*U + a - pad for U in [lo, lo + count); they are reached through the `taps`
// window taps p = a + s*i.
struct PhaseDim {
    int taps, lo, count;
};
PhaseDim phase_dim(int extent, int k, int s, int pad, int a)
{
    PhaseDim d;
    d.taps = a < k ? (k - a + s - 1) / s : 0;
    d.lo = pad - a > 0 ? (pad - a + s - 1) / s : 0;
    const int top = extent - 1 + pad - a;  // s*U <= top
    const int hi = top >= 0 ? top / s : -1;
    d.count = hi - d.lo + 1 > 0 ? hi - d.lo + 1 : 0;
    return d;
}
// phase (a,b) as a forward convolution for the tuned kernels (16-bit or fp32)
ConvShape bwd_input_phase_shape(const ConvShape& s, const PhaseDim& ph, const PhaseDim& pw, int a,
                                int b)
{
    ConvShape f{s.N, s.Ho, s.Wo, s.M, s.C, ph.taps, pw.taps, 1, ph.taps - 1 - ph.lo,
                s.D0, s.D1, s.D3, s.D2, ph.count, pw.count, s.dtype};
    f.out16 = s.out16;
    same_small_tiles(f, s);
    f.in_gradient = true;
    f.pad_w_set = true;
    f.pad_w = pw.taps - 1 - pw.lo;
    f.out_view = true;
    const long long pix = (long long)s.C * s.D0 * s.D1 * s.D2;
    f.out_sn = (long long)s.H * s.W * pix;
    f.out_sx = (long long)s.stride * s.W * pix;
    f.out_sy = (long long)s.stride * pix;
    f.out_base = ((long long)(s.stride * ph.lo + a - s.pad) * s.W + (s.stride * pw.lo + b - s.pad)) * pix;
    f.out_alloc = (long long)s.in_elems();
    return f;
}
// which tuned kernel runs a phase: 16 = the 256x256-tile 16-bit kernel, 32 = the lane-per-row
// kernel (fp32, or 16-bit shapes the other one does not take), 0 = neither fits or fills the chip
int phase_kernel(const ConvShape& f)
{
    if (!mfma_supported(f)) return 0;
    if (f.dtype != 0 && mfma_tuned16_supported(f) &&
        (long long)f.N * f.Ho * f.Wo * f.D1 >= 256LL * 128)
        return 16;
    // the lane-per-row kernel with an unsplit K loop (an output view takes no partial sums)
    if (mfma_dma32_supported(f) && igemm32_dma_preferred(f)) return 32;
    return 0;
}

// 16-bit layers with capsule columns of 4 elements: the phases that run on the lane-per-row
// kernel read the output gradient with its channels paired; it is paired once for all of them
bool phases_pair_dout(const ConvShape& s) { return s.dtype != 0 && s.D3 == 4 && s.M % 2 == 0; }

// a phase's kernel tensor read in place: the convolution's input channels are the layer's output
// channels, its contracted capsule index the layer's d3
void view_phase_kernel(const ConvShape& s, const PhaseDim& ph, const PhaseDim& pw, int a, int b, ConvShape& f)
{
    const long long sD0 = (long long)s.D2 * s.D3, sM = sD0 * s.D0, sC = sM * s.M, sQ = sC * s.C, sP = sQ * s.kw;
    f.kernel_view = true;
    f.k_base = (long long)(a + s.stride * (ph.taps - 1)) * sP + (long long)(b + s.stride * (pw.taps - 1)) * sQ;
    f.k_sp = -s.stride * sP;
    f.k_sq = -s.stride * sQ;
    f.k_sc = sM;
    f.k_sm = sC;
    f.k_sd0 = sD0;
    f.k_sd2 = 1;
    f.k_sd3 = s.D3;
}

// The input gradient as phases in one launch of the small-tile kernel (any window, padding and
// stride up to 4; a stride of 1 is one phase).  Returns their number, 0 if there are too many.
constexpr int kMaxPhases = 16;
static_assert(kMaxPhases <= MAX_REPACK_VIEWS);
int bwd_input_phases(const ConvShape& s, ConvShape (&f)[kMaxPhases])
{
    if (s.stride > 4) return 0;
    int n = 0;
    for (int a = 0; a < s.stride; ++a)
        for (int b = 0; b < s.stride; ++b) {
            const PhaseDim ph = phase_dim(s.H, s.kh, s.stride, s.pad, a);
            const PhaseDim pw = phase_dim(s.W, s.kw, s.stride, s.pad, b);
            if (ph.count == 0 || pw.count == 0) continue;
            ConvShape& g = f[n++];
            g = bwd_input_phase_shape(s, ph, pw, a, b);
            view_phase_kernel(s, ph, pw, a, b, g);
        }
    return n;
}

// every phase that has both pixels and taps must fit a tuned kernel and fill the chip
bool bwd_input_as_phases(const ConvShape& s)
{
    if (s.stride == 1 || s.stride > 4) return false;
    for (int a = 0; a < s.stride; ++a)
        for (int b = 0; b < s.stride; ++b) {
            const PhaseDim ph = phase_dim(s.H, s.kh, s.stride, s.pad, a);
            const PhaseDim pw = phase_dim(s.W, s.kw, s.stride, s.pad, b);
            if (ph.count == 0 || pw.count == 0 || ph.taps == 0 || pw.taps == 0) continue;
            const ConvShape f = bwd_input_phase_shape(s, ph, pw, a, b);
            if (phase_kernel(f) == 0) return false;
        }
    return true;
}

// The phases that have both pixels and taps, for the tuned kernels, and where in the scratch their repacked kernels lie
// when one launch packs them all (`together`: those of a 16-bit layer that fit the scratch side by side; nearly always,
// not where few columns are padded to twice their number), else each phase's lies at `paired`, packed before it.
// One launch against one per phase: 18 random layers 0.85 .. 0.99 of the time, 0.95 on average (108 images of 22x22,
// 5 -> 3 channels of 8x8 capsules, 49.2 -> 41.8 us); 128 images of 28x28, 64 -> 64 channels of 8x8, 1014 -> 1007.
struct PhaseRun {
    int n;
    ConvShape f[kMaxPhases];
    MfmaKernel which[kMaxPhases];
    RepackLayout layout[kMaxPhases];
    size_t at[kMaxPhases];
    size_t paired;  // bytes of the output gradient with its channels paired, at the scratch's start
    bool together;
};
void bwd_input_phase_run(const ConvShape& s, size_t scratch_bytes, PhaseRun& r)
{
    r.paired = phases_pair_dout(s) ? align256(s.out_elems() * elem_bytes(s)) : 0;
    r.n = 0;
    for (int a = 0; a < s.stride; ++a)
        for (int b = 0; b < s.stride; ++b) {
            const PhaseDim ph = phase_dim(s.H, s.kh, s.stride, s.pad, a);
            const PhaseDim pw = phase_dim(s.W, s.kw, s.stride, s.pad, b);
            if (ph.count == 0 || pw.count == 0 || ph.taps == 0 || pw.taps == 0) continue;
            // the phase's kernel Kab[i'][j'][m][c][d0][d3][d2] =
            // K[a + s*(taps_h-1-i')][b + s*(taps_w-1-j')][c][m][d0][d2][d3] is read in place:
            // the repack pass of the convolution takes it through strides
            ConvShape& f = r.f[r.n];
            f = bwd_input_phase_shape(s, ph, pw, a, b);
            view_phase_kernel(s, ph, pw, a, b, f);
            const bool lane_per_row = phase_kernel(f) == 32;
            f.in_paired = lane_per_row && r.paired > 0;
            r.which[r.n++] = lane_per_row ? MfmaKernel::Dma32 : MfmaKernel::Tuned16;
        }
    size_t at = r.paired;
    r.together = r.n > 1;
    for (int i = 0; i < r.n && r.together; ++i) {
        r.layout[i] = mfma_repack_layout(r.f[i], r.which[i]);
        r.at[i] = at;
        const size_t bytes = align256(r.layout[i].bytes);
        r.together = bytes != 0 && bytes <= scratch_bytes - at;
        at += bytes;
    }
}

// zero the pixels (n, h0 + i*sh, w0 + j*sw), i < nh, j < nw, of a tensor [N][H][W][pix] of fp32
// (T = float) or 16-bit (T = unsigned short) elements
template <typename T>
__global__ __launch_bounds__(256) void zero_pixels_kernel(T* __restrict__ out, int H, int W,
                                                          long long pix, int h0, int sh, int nh,
                                                          int w0, int sw, int nw, size_t total)
{
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= total) return;
    size_t r = id;
    const long long e = (long long)(r % pix); r /= pix;
    const int j = (int)(r % nw); r /= nw;
    const int i = (int)(r % nh);
    const long long n = (long long)(r / nh);
    out[((n * H + h0 + (long long)i * sh) * W + w0 + (long long)j * sw) * pix + e] = T(0);
}

// fully-connected layer: one output pixel, the window is the whole unpadded image
bool bwd_input_as_fc(const ConvShape& s)
{
    return s.Ho == 1 && s.Wo == 1 && s.pad == 0 && s.kh == s.H && s.kw == s.W;
}
ConvShape bwd_input_fc_shape(const ConvShape& s)
{
    // input G [N][1][1][M][D0][D1][D3], kernel [1][1][M][(h,w,c)][D0][D3][D2] -> dI [N][(h,w,c)][D0][D1][D2]
    ConvShape f{s.N, 1, 1, s.M, s.kh * s.kw * s.C, 1, 1, 1, 0, s.D0, s.D1, s.D3, s.D2, 1, 1,
                s.dtype};
    f.out16 = s.out16;
    same_small_tiles(f, s);
    f.in_gradient = true;
    return f;
}
// dI as a forward convolution of the (spread-out) G with the flipped, transposed kernel
bool bwd_input_as_conv(const ConvShape& s) { return s.kh == s.kw && s.pad <= s.kh - 1; }
ConvShape bwd_input_conv_shape(const ConvShape& s)
{
    // input Gs [N][Hs][Ws][M][D0][D1][D3], kernel K' [kh][kw][M][C][D0][D3][D2] -> dI [N][H][W][C][D0][D1][D2]
    ConvShape f{s.N, spread_h(s), spread_w(s), s.M, s.C, s.kh, s.kw, 1, s.kh - 1 - s.pad,
                s.D0, s.D1, s.D3, s.D2, s.H, s.W, s.dtype};
    f.out16 = s.out16;
    same_small_tiles(f, s);
    f.in_gradient = true;
    return f;
}
// ... with the kernel tensor read in place
void view_kernel(const ConvShape& s, ConvShape& f)
{
    f.kernel_view = true;
    f.k_sc = (long long)s.D2 * s.D3 * s.D0;
    f.k_sm = f.k_sc * s.M;
    f.k_sd0 = (long long)s.D2 * s.D3;
    f.k_sd2 = 1;
    f.k_sd3 = s.D3;
}
void view_flipped_kernel(const ConvShape& s, ConvShape& f)
{
    view_kernel(s, f);
    const long long sQ = f.k_sm * s.C, sP = sQ * s.kw;
    f.k_base = (long long)(s.kh - 1) * sP + (long long)(s.kw - 1) * sQ;
    f.k_sp = -sP;
    f.k_sq = -sQ;
}

// fp32: against the estimates of what would run, the spread-out gradient's zeros counted in (20 random strided
// layers: 19 of them 0.15 .. 0.85 times the time, one whose phases fill the bf16 kernel's tiles stays there)
bool mid_preferred32(const ConvShape& s, const BwdInputPlan& plan, const ConvShape* f, int n, double us)
{
    double other = 0;
    if (plan.form == BwdInputPlan::Phases) {
        for (int i = 0; i < n; ++i)  // (the phases' launches overlap: 9 us less than their calls' times)
            if (f[i].kh * f[i].kw > 0) other += igemm32_us(f[i], MfmaKernel::Dma32) - 9.0;
    } else {
        const ConvShape c = bwd_input_conv_shape(s);
        other = 8.0 + igemm32_us(c, plan.fwd.kernel == MfmaKernel::Auto ? mfma_auto_kernel(c) : plan.fwd.kernel);
    }
    return us < 0.75 * other;
}

// Strided layers, and the windows and paddings that the convolution form does not cover, on the small-tile
// kernel: always where `dout` would be spread out (16-bit; s^2 times the work) or gathered element by element
// (220 random layers, none slower), else
// where one launch is estimated a quarter faster than the phases' launches on the tuned kernels.  These overlap (9 us less than
// their calls' times), and the phases of one launch each read `dout`, 5.9 TB/s, which the estimate of one convolution
// leaves out: 37 strided 16-bit layers of four phases 20 % off, 35 % without; 11 of them go, for 0.3 .. 1.0 of the time
// (without both and at 30 %: 22, of which 16 -> 56 channels of 4x8 . 8x16, N = 101, 34x34, and two others 1.5 times the time).
// Stride 1 otherwise is a convolution whose kernel the forward pass's rules pick.
MidPick bwd_input_on_mid(const ConvShape& s, const BwdInputPlan& plan, const ConvShape* f, int n, size_t room)
{
    if (n == 0 || !igemm_mid_eligible(f, n, s.kernel_elems())) return {};
    const MidEstimate e = igemm_mid_best(f, n, room);
    bool take = true;
    if (s.mid_use == 2) {
    } else if (s.dtype == 0 && plan.form != BwdInputPlan::Gather) {
        take = mid_preferred32(s, plan, f, n, e.us);
    } else if (plan.form == BwdInputPlan::Phases) {
        double other = 9.0, reads = 0;
        for (int i = 0; i < n; ++i) {
            if (f[i].kh * f[i].kw == 0) continue;
            other += igemm16_tuned_us(f[i], phase_kernel(f[i]) == 16 ? MfmaKernel::Tuned16 : MfmaKernel::Dma32) - 9.0;
            reads += 1.0;
        }
        const double mb = 2e-6 * (double)s.out_elems(), out_mb = (s.out16 ? 2e-6 : 4e-6) * (double)s.in_elems();
        take = e.us + 0.17 * reads * mb + 0.03 * out_mb < 0.75 * other;
    }
    return take ? e.pick : MidPick{};
}

bool phases_may_run_on_mid(const ConvShape& s, const BwdInputPlan& plan)
{
    return plan.form != BwdInputPlan::FullyConnected && (s.stride > 1 || plan.form == BwdInputPlan::Gather);
}
size_t small_tile_room(const ConvShape& s, size_t need, size_t workspace_bytes)
{
    return s.mid_use == 2 ? workspace_bytes : need;
}

// dK as a forward convolution of the re-laid-out input with the (spread-out) output gradient
// as the window
ConvShape bwd_kernel_conv_shape(const ConvShape& s)
{
    // input I' [C][H][W][N][D0][D2][D1], kernel G' [Hs][Ws][N][M][D0][D1][D3] -> [C][kh][kw][M][D0][D2][D3]
    ConvShape f{s.C, s.H, s.W, s.N, s.M, spread_h(s), spread_w(s), 1, s.pad,
                s.D0, s.D2, s.D1, s.D3, s.kh, s.kw, s.dtype};
    same_small_tiles(f, s);
    return f;
}

}  // namespace

BwdInputPlan bwd_input_plan(const ConvShape& s)
{
    BwdInputPlan plan{BwdInputPlan::Gather, {}, 0};
    const size_t kbytes = align256(s.kernel_elems() * elem_bytes(s));
    if (bwd_input_as_fc(s)) {
        const ConvShape f = bwd_input_fc_shape(s);
        plan.form = BwdInputPlan::FullyConnected;
        plan.fwd = forward_choice(f);
        plan.bytes = kbytes + forward_choice_bytes(f, plan.fwd);
    } else if (bwd_input_as_phases(s)) {
        plan.form = BwdInputPlan::Phases;
        size_t fwd = 0;
        for (int a = 0; a < s.stride; ++a)
            for (int b = 0; b < s.stride; ++b) {
                const PhaseDim ph = phase_dim(s.H, s.kh, s.stride, s.pad, a);
                const PhaseDim pw = phase_dim(s.W, s.kw, s.stride, s.pad, b);
                if (ph.count == 0 || pw.count == 0 || ph.taps == 0 || pw.taps == 0) continue;
                ConvShape f = bwd_input_phase_shape(s, ph, pw, a, b);
                f.in_paired = phases_pair_dout(s);
                const size_t need = mfma_workspace_bytes(f);
                if (need > fwd) fwd = need;
            }
        // (the kernel tensor's size and the largest phase's scratch: room for all phases' repacked kernels side by
        // side, padding apart)
        plan.bytes = kbytes + fwd + (phases_pair_dout(s) ? align256(s.out_elems() * elem_bytes(s)) : 0);
    } else if (bwd_input_as_conv(s)) {
        const ConvShape f = bwd_input_conv_shape(s);
        plan.form = BwdInputPlan::Convolution;
        plan.fwd = forward_choice(f);
        plan.bytes = kbytes + (s.stride > 1 ? align256(spread_elems(s) * elem_bytes(s)) : 0) +
                     forward_choice_bytes(f, plan.fwd);
    }
    return plan;
}

size_t bwd_kernel_workspace_bytes(const ConvShape& s)
{
    if (wgrad16_eligible(s)) return wgrad16_workspace_bytes(s);
    if (wgrad32_eligible(s)) return wgrad32_workspace_bytes(s);
    const ConvShape f = bwd_kernel_conv_shape(s);
    return align256(s.in_elems() * elem_bytes(s)) + align256(spread_elems(s) * elem_bytes(s)) +
           align256(s.kernel_elems() * sizeof(float)) + forward_choice_bytes(f, forward_choice(f));
}

RouteInfo bwd_input_route(const ConvShape& s, const BwdInputPlan& plan, size_t workspace_bytes)
{
    MidPick pick;
    if (phases_may_run_on_mid(s, plan)) {
        ConvShape f[kMaxPhases];
        const int n = bwd_input_phases(s, f);
        pick = bwd_input_on_mid(s, plan, f, n, small_tile_room(s, plan.bytes, workspace_bytes));
        if (plan.form == BwdInputPlan::Gather) pick.nsplit = 1;
    }
    if (!pick && (plan.form == BwdInputPlan::FullyConnected || plan.form == BwdInputPlan::Convolution)) {
        const bool fc = plan.form == BwdInputPlan::FullyConnected;
        ConvShape f = fc ? bwd_input_fc_shape(s) : bwd_input_conv_shape(s);
        if (plan.fwd.takes_kernel_view && fc) view_kernel(s, f);
        if (plan.fwd.takes_kernel_view && !fc) view_flipped_kernel(s, f);
        const size_t used = plan.bytes - forward_choice_bytes(f, plan.fwd);
        pick = forward_small_tiles(f, plan.fwd, workspace_bytes > used ? workspace_bytes - used : 0);
    }
    return {pick.tile, pick.nsplit, plan.form};
}

bool bwd_input_repacks_together(const ConvShape& s, const BwdInputPlan& plan)
{
    if (plan.form != BwdInputPlan::Phases || bwd_input_route(s, plan, plan.bytes).tile >= 0) return false;
    PhaseRun r;
    bwd_input_phase_run(s, plan.bytes, r);
    return r.together;
}

RouteInfo bwd_kernel_route(const ConvShape& s, size_t need, size_t workspace_bytes)
{
    const MidPick pick = wgrad_mid_choice(s, small_tile_room(s, need, workspace_bytes));
    return {pick.tile, pick.nsplit, wgrad16_eligible(s) ? 16 : wgrad32_eligible(s) ? 32 : 1};
}

// `din` holds fp32 elements, or with s.out16 set 16-bit elements of that kind (every route's
// convolution shape carries s.out16 on, so its kernels round once at their stores).
int launch_bwd_input(const ConvShape& s, const BwdInputPlan& plan, const void* dout, const void* kernel,
                     float* din, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const int eb = elem_bytes(s);
    const long long sD3 = 1, sD2 = s.D3, sD0 = (long long)s.D2 * s.D3, sM = sD0 * s.D0,
                    sC = sM * s.M, sQ = sC * s.C, sP = sQ * s.kw;
    if (plan.form == BwdInputPlan::FullyConnected) {
        char* ws = static_cast<char*>(workspace);
        const size_t used = align256(s.kernel_elems() * eb);
        // K2[m][(h,w,c)][d0][d3][d2] = K[h][w][c][m][d0][d2][d3]; (h,w,c) is one index of stride sC
        ConvShape f = bwd_input_fc_shape(s);
        if (plan.fwd.takes_kernel_view) {
            view_kernel(s, f);  // ((h,w,c) is one index of stride k_sm)
            return forward_run(f, plan.fwd, dout, kernel, din, ws + used, workspace_bytes - used, stream);
        }
        const Permute7 pm = gather_into_dense(
            {1, 1, s.M, (long long)s.kh * s.kw * s.C, s.D0, s.D3, s.D2},
            {0, 0, sM, sC, sD0, sD3, sD2}, 0);
        hipError_t err = launch_permute(kernel, ws, pm, eb, stream);
        if (err != hipSuccess) return status_from_hip(err);
        return forward_run(f, plan.fwd, dout, ws, din, ws + used, workspace_bytes - used, stream);
    }
    if (phases_may_run_on_mid(s, plan)) {
        ConvShape f[kMaxPhases];
        const int n = bwd_input_phases(s, f);
        // (in the place of the gather kernel: like it, no tap outside the image)
        if (const MidPick pick = bwd_input_on_mid(s, plan, f, n, small_tile_room(s, plan.bytes, workspace_bytes)))
            return status_from_hip(launch_igemm_mid(f, n, s.kernel_elems(), pick, dout, kernel, din, workspace,
                                                    stream, plan.form == BwdInputPlan::Gather));
    }
    if (plan.form == BwdInputPlan::Phases) {
        char* ws = static_cast<char*>(workspace);
        const long long pix = (long long)s.C * s.D0 * s.D1 * s.D2;
        PhaseRun r;
        bwd_input_phase_run(s, plan.bytes, r);
        if (r.paired > 0) {
            const hipError_t err = launch_pair_channels(dout, ws, (size_t)s.N * s.Ho * s.Wo, s.M,
                                                        s.D0 * s.D1, stream);
            if (err != hipSuccess) return status_from_hip(err);
        }
        for (int a = 0; a < s.stride; ++a)
            for (int b = 0; b < s.stride; ++b) {
                const PhaseDim ph = phase_dim(s.H, s.kh, s.stride, s.pad, a);
                const PhaseDim pw = phase_dim(s.W, s.kw, s.stride, s.pad, b);
                if (ph.count == 0 || pw.count == 0) continue;  // no pixel of dI in this phase
                if (ph.taps > 0 && pw.taps > 0) continue;
                // pixels no window reaches
                const int h0 = s.stride * ph.lo + a - s.pad, w0 = s.stride * pw.lo + b - s.pad;
                const size_t total = (size_t)s.N * ph.count * pw.count * pix;
                const size_t blocks = (total + 255) / 256;
                if (blocks > 0x7fffffffULL) return status_from_hip(hipErrorInvalidValue);
                if (s.out16 != 0)
                    zero_pixels_kernel<unsigned short><<<(unsigned)blocks, 256, 0, stream>>>(
                        reinterpret_cast<unsigned short*>(din), s.H, s.W, pix, h0, s.stride,
                        ph.count, w0, s.stride, pw.count, total);
                else
                    zero_pixels_kernel<float><<<(unsigned)blocks, 256, 0, stream>>>(
                        din, s.H, s.W, pix, h0, s.stride, ph.count, w0, s.stride, pw.count,
                        total);
                const hipError_t err = hipGetLastError();
                if (err != hipSuccess) return status_from_hip(err);
            }
        if (r.together) {
            void* kp[kMaxPhases];
            for (int i = 0; i < r.n; ++i) kp[i] = ws + r.at[i];
            const hipError_t err = launch_repack_views(r.f, r.layout, kp, r.n, kernel, stream);
            if (err != hipSuccess) return status_from_hip(err);
        }
        for (int i = 0; i < r.n; ++i) {
            const void* g = r.f[i].in_paired ? ws : dout;
            char* own = ws + r.paired;
            const size_t own_bytes = workspace_bytes - r.paired;
            const int rc =
                r.together ? status_from_hip(launch_mfma_repacked(r.f[i], g, ws + r.at[i], din, stream, r.which[i]))
                : r.which[i] == MfmaKernel::Dma32 ? forward_tuned32(r.f[i], g, kernel, din, own, own_bytes, stream)
                                                  : forward_tuned16(r.f[i], g, kernel, din, own, own_bytes, stream);
            if (rc != 0) return rc;
        }
        return 0;
    }
    if (plan.form == BwdInputPlan::Convolution) {
        char* ws = static_cast<char*>(workspace);
        const void* kflip = ws;
        size_t used = align256(s.kernel_elems() * eb);
        // K'[p'][q'][m][c][d0][d3][d2] = K[kh-1-p'][kw-1-q'][c][m][d0][d2][d3]
        ConvShape f = bwd_input_conv_shape(s);
        hipError_t err = hipSuccess;
        if (plan.fwd.takes_kernel_view) {  // read in place
            view_flipped_kernel(s, f);
            kflip = kernel;
        } else {
            const Permute7 pm = gather_into_dense({s.kh, s.kw, s.M, s.C, s.D0, s.D3, s.D2},
                                                  {-sP, -sQ, sM, sC, sD0, sD3, sD2},
                                                  (long long)(s.kh - 1) * sP + (long long)(s.kw - 1) * sQ);
            err = launch_permute(kernel, ws, pm, eb, stream);
            if (err != hipSuccess) return status_from_hip(err);
        }
        const void* g = dout;
        if (s.stride > 1) {
            // Gs[n][x*s][y*s] = G[n][x][y], zero elsewhere; a pixel (M capsules) moves as one run
            void* gs = ws + used;
            const size_t gbytes = align256(spread_elems(s) * eb);
            used += gbytes;
            err = launch_fill_zero(gs, gbytes, stream);
            if (err != hipSuccess) return status_from_hip(err);
            const long long pix = (long long)s.M * s.D0 * s.D1 * s.D3;
            Permute7 sp{};
            const long long dim[7] = {1, 1, 1, s.N, s.Ho, s.Wo, pix};
            const long long ss[7] = {0, 0, 0, (long long)s.Ho * s.Wo * pix, s.Wo * pix, pix, 1};
            const long long ds[7] = {0, 0, 0, (long long)spread_h(s) * spread_w(s) * pix,
                                     (long long)s.stride * spread_w(s) * pix, s.stride * pix, 1};
            for (int k = 0; k < 7; ++k) {
                sp.dim[k] = dim[k];
                sp.src_stride[k] = ss[k];
                sp.dst_stride[k] = ds[k];
            }
            err = launch_permute(dout, gs, sp, eb, stream);
            if (err != hipSuccess) return status_from_hip(err);
            g = gs;
        }
        return forward_run(f, plan.fwd, g, kflip, din, ws + used, workspace_bytes - used, stream);
    }
    const size_t total = s.in_elems();
    hipError_t err;
    if (s.dtype == 0)
        err = launch_1d(bwd_input_direct_kernel<float>, total, stream, (const float*)dout,
                        (const float*)kernel, din, s);
    else if (s.dtype == 1)
        err = launch_1d(bwd_input_direct_kernel<__hip_bfloat16>, total, stream,
                        (const __hip_bfloat16*)dout, (const __hip_bfloat16*)kernel, din, s);
    else
        err = launch_1d(bwd_input_direct_kernel<__half>, total, stream, (const __half*)dout,
                        (const __half*)kernel, din, s);
    return status_from_hip(err);
}

int launch_bwd_kernel(const ConvShape& s, size_t need, const void* input, const void* dout, float* dkernel,
                      void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (const MidPick pick = wgrad_mid_choice(s, small_tile_room(s, need, workspace_bytes)))
        return status_from_hip(launch_wgrad_mid(s, pick, input, dout, dkernel, workspace, stream));
    if (wgrad16_eligible(s))
        return status_from_hip(launch_wgrad16(s, input, dout, dkernel, workspace, stream));
    if (wgrad32_eligible(s))
        return status_from_hip(launch_wgrad32(s, input, dout, dkernel, workspace, stream));
    const int eb = elem_bytes(s);
    char* ws = static_cast<char*>(workspace);
    void* in_t = ws;
    size_t used = align256(s.in_elems() * eb);
    void* g_t = ws + used;
    const size_t gbytes = align256(spread_elems(s) * eb);
    used += gbytes;
    float* dk_t = reinterpret_cast<float*>(ws + used);
    used += align256(s.kernel_elems() * sizeof(float));
    // I'[c][h][w][n][d0][d2][d1] = I[n][h][w][c][d0][d1][d2]
    {
        const long long sD2 = 1, sD1 = s.D2, sD0 = (long long)s.D1 * s.D2, sC = sD0 * s.D0,
                        sW = sC * s.C, sH = sW * s.W, sN = sH * s.H;
        const Permute7 pm = gather_into_dense({s.C, s.H, s.W, s.N, s.D0, s.D2, s.D1},
                                              {sC, sH, sW, sN, sD0, sD2, sD1}, 0);
        hipError_t err = launch_permute(input, in_t, pm, eb, stream);
        if (err != hipSuccess) return status_from_hip(err);
    }
    // G'[x*s][y*s][n][m][d0][d1][d3] = G[n][x][y][m][d0][d1][d3], zero elsewhere
    {
        if (s.stride > 1) {
            hipError_t err = launch_fill_zero(g_t, gbytes, stream);
            if (err != hipSuccess) return status_from_hip(err);
        }
        const long long caps = (long long)s.D0 * s.D1 * s.D3, sM = caps, sY = sM * s.M,
                        sX = sY * s.Wo, sN = sX * s.Ho;
        Permute7 pm = gather_into_dense({s.Ho, s.Wo, s.N, s.M, s.D0, s.D1, s.D3},
                                        {sX, sY, sN, sM, (long long)s.D1 * s.D3, s.D3, 1}, 0);
        const long long pix = (long long)s.N * s.M * caps;  // one window tap of G'
        pm.dst_stride[0] = (long long)s.stride * spread_w(s) * pix;
        pm.dst_stride[1] = (long long)s.stride * pix;
        hipError_t err = launch_permute(dout, g_t, pm, eb, stream);
        if (err != hipSuccess) return status_from_hip(err);
    }
    const ConvShape f = bwd_kernel_conv_shape(s);
    const int rc = forward_run(f, forward_choice(f), in_t, g_t, dk_t, ws + used, workspace_bytes - used, stream);
    if (rc != 0) return rc;
    // dK[p][q][c][m][d0][d2][d3] = dK'[c][p][q][m][d0][d2][d3]
    const long long caps = (long long)s.D0 * s.D2 * s.D3, sM = caps, sQ = sM * s.M,
                    sP = sQ * s.kw, sC = sP * s.kh;
    const Permute7 pm = gather_into_dense({s.kh, s.kw, s.C, s.M, s.D0, s.D2, s.D3},
                                          {sP, sQ, sC, sM, (long long)s.D2 * s.D3, s.D3, 1}, 0);
    return status_from_hip(launch_permute(dk_t, dkernel, pm, 4, stream));
}

}  // namespace capscaps
