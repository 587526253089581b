// 16-bit matrix-core kernel of the capsule convolution forward pass, one tile row per lane, with
// direct-to-LDS copies.  Same implicit GEMM as the other igemm kernels (rows (pixel,d1), columns
// (m,d3), K = (tap, c, d2); paper Algorithm 2), for any D1 and D3: non-square and vector
// capsules, which the 256x256-tile 16-bit kernel does not take, and 4x4 capsules.  This file
// also holds the tile and split decisions of the fp32 kernel of the same row layout
// (igemm32_split.hip).
//
// Unit of data movement: a 16-byte LDS slot holding 8 consecutive d2 of one capsule row ("chunk");
// lengths and offsets are counted in units of 4 bytes ("floats": a capsule row of 8, 16 or 32
// halves is one of 4, 8 or 16 of them).  A chunk pair feeds one MFMA 32x32x16 per tile.
//
// Tile: 64*NW rows x 32*TN columns; wave w copies and contracts rows 64w..64w+63 (two MFMA
// row tiles) against all TN column tiles.  Lane i of a wave copies row 64w+i: its byte offset,
// with the out-of-range mark where the current tap falls into the padding, sits in one VGPR
// and is refreshed once per stage from a per-lane bit mask over the taps; everything else
// (tap, channel group, chunk) is a scalar offset.  K runs channel group outermost, tap inside,
// 2 or 4 chunks per stage, ring of 3 or 4 LDS stages, one barrier per stage; the K loop can be
// split over blocks (partial sums are reduced in a fixed order by the caller's reduce kernel).
//
// Rows of 4 halves (4x4 capsules) no 16-byte copy can stage as they lie in memory: the 8 K values
// a 16-bit matrix instruction takes per lane are the rows of two channels, 32 bytes apart.  A
// pre-pass (pair_channels_kernel, at HBM speed) writes the input with channels paired,
// [pixel][c/2][d0][d1][c%2][d2]; that is a layer with half the channels and rows of 4 "floats", so
// every offset and copy of this kernel stays as it is.
#include <hip/hip_runtime.h>

#include <cmath>

#include "igemm_common.h"
#include "lds_dma.h"

namespace capscaps {
namespace {

// KCH chunks per row and stage, ring of NB stages.  Small stages (2 chunks) halve the LDS
// footprint of a workgroup, so that more of them share a CU and one wave's copies and waits run
// under the others' MFMAs; they need capsule rows of at most 2 chunks.  With up to three column
// tiles the kernel is compiled for four waves per SIMD (126 registers: the accumulators and a
// small stage's operands) and takes a ring of three stages, so that four four-wave workgroups
// share a CU; elsewhere the compiler's own register budget and the deeper ring of the small stages.
constexpr int waves_per_simd(int tn, int nw, int kch) { return nw == 4 && tn <= 3 && kch == 2 ? 4 : 1; }
// The 16-bit-output variants are held to the waves per SIMD their fp32-output twins reach by
// themselves (32 TN accumulator registers and about 30 others): left alone, the compiler reads
// all accumulators out for the rounding at once (146 registers more with four column tiles), one
// wave per SIMD remains, and a layer of 64 channels of 4x4 capsules runs 35 % slower with 16-bit
// than with fp32 output.
constexpr int waves_per_simd_out16(int tn, int nw, int kch)
{
    return waves_per_simd(tn, nw, kch) > 1 ? waves_per_simd(tn, nw, kch) : tn == 1 ? 6 : tn == 2 ? 4 : 3;
}
constexpr int ring_depth(int kch, int tn, int nw) { return kch == 2 && waves_per_simd(tn, nw, kch) == 1 ? 4 : 3; }

// OUT16: the output has the operands' type, rounded at the store.
template <typename Tag, int TN, int NW, int KCH, bool OUT16 = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(OUT16 ? waves_per_simd_out16(TN, NW, KCH) : waves_per_simd(TN, NW, KCH)))) void igemm32_dma_kernel(const Dma32Params P)
{
    // a compile-time constant: with the choice made at run time the register allocator fails
    // to keep the copies' buffer descriptors in scalar registers
    constexpr int o16 = !OUT16 ? 0 : std::is_same<Tag, f16_tag>::value ? 2 : 1;
    constexpr int CW = 4;  // "floats" per chunk
    constexpr int NB = ring_depth(KCH, TN, NW);
    constexpr int BM = 64 * NW, BN = 32 * TN, BNL = (BN + 63) / 64 * 64, TM = 2;
    constexpr int A_BYTES = KCH * BM * 16, B_BYTES = KCH * BNL * 16;
    constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    constexpr int NBC = KCH * BNL / 64;  // kernel-side copies per stage, all waves
    constexpr int BPW = NBC / NW;        // ... per wave
    static_assert(NBC % NW == 0, "kernel copies divide evenly over the waves");
    constexpr int NCOPY = KCH + BPW;     // copies per wave and stage
    constexpr int OOB = (int)0x80000000u;
    // at a barrier the copies of the NB-2 most recent stages may still be in flight
    constexpr int KEEP = (NB - 2) * NCOPY;
    static_assert(KEEP < 64, "vmcnt is a 6-bit counter");
    constexpr int VMCNT_KEEP = 0x0F70 | (KEEP & 15) | ((KEEP >> 4) << 14);

    extern __shared__ char smem[];

    // ---- tile: column tiles fastest, then row tiles, leading capsule index, K split
    int L = blockIdx.x;
    int col_tile, row_tile, d0, split;
    if (P.xcd_span > 0) {
        // the D0 tiles of one (row tile, column tile) read the same input lines and write into
        // the same output lines: they run at the same time on one XCD and meet in its L2
        if (L < P.xcd_span) L = (L & 7) * (P.xcd_span >> 3) + (L >> 3);
        d0 = L % P.D0;
        int rest = L / P.D0;
        col_tile = rest % P.col_tiles;
        rest /= P.col_tiles;
        row_tile = rest % P.row_tiles;
        split = rest / P.row_tiles;
    } else {
        col_tile = L % P.col_tiles;
        int rest = L / P.col_tiles;
        row_tile = rest % P.row_tiles;
        rest /= P.row_tiles;
        d0 = rest % P.D0;
        split = rest / P.D0;
    }

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, lr = lane & 31;
    const long long row0 = (long long)row_tile * BM;
    const int col0 = col_tile * BN;

    // ---- this lane's row: byte offset of its capsule row in the window's first input pixel,
    // relative to the first image the tile touches, and the bit mask of taps that read a real
    // input pixel
    const int hw = P.Ho * P.Wo;
    const long long n_first = (row0 / P.D1) / hw;
    const long long img_bytes = (long long)P.H * P.W * P.pixsz * 4;
    const int pix_bytes = (int)(P.pixsz * 4);
    // Lane offsets must not be negative (the hardware adds lane and scalar offset without
    // wrapping), but a window's first pixel may lie in the padding: the descriptor's base is
    // moved back by the largest such distance and every lane offset forward by the same.
    // Nothing is read below the tensor: only in-range taps are ever addressed.
    const int bias = ((P.pad > 0 ? P.pad : 0) * P.W + (P.pad_w > 0 ? P.pad_w : 0)) * pix_bytes;
    const char* in_base = static_cast<const char*>(P.in) + n_first * img_bytes - bias;
    int row_off;
    unsigned long long tap_ok = 0;
    {
        const long long rg = row0 + 64 * wave + lane;
        const bool exists = rg < P.rows;
        const long long rr = exists ? rg : row0;
        const long long pixel = rr / P.D1;
        const int d1 = (int)(rr % P.D1);
        const int n_rel = (int)(pixel / hw - n_first);
        const int rem = (int)(pixel % hw);
        const int x = rem / P.Wo, y = rem - x * P.Wo;
        const int ih0 = x * P.stride - P.pad, iw0 = y * P.stride - P.pad_w;
        row_off = (int)((((long long)n_rel * P.H + ih0) * P.W + iw0) * pix_bytes) +
                  (d0 * P.D1 + d1) * P.D2 * 4 + bias;
        if (exists) {
            int t = 0;
            for (int p = 0; p < P.kh; ++p)
                for (int q = 0; q < P.kw; ++q, ++t)
                    if ((unsigned)(ih0 + p) < (unsigned)P.H && (unsigned)(iw0 + q) < (unsigned)P.W)
                        tap_ok |= 1ull << t;
        }
    }
    long long in_left = P.in_bytes - n_first * img_bytes + bias;
    if (in_left > 0x7fffffffLL) in_left = 0x7fffffffLL;
    const rsrc_t rs_in = make_rsrc(in_base, (unsigned)in_left);
    rsrc_t rs_none = rs_in;  // nothing addressable: every lane stores zeros
    rs_none[2] = 0;
    const rsrc_t rs_kp = make_rsrc(P.kp, (unsigned)P.kp_bytes);
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;

    // ---- K loop state of the next stage to copy (all scalar)
    const int st_begin = split * P.stages_per_split;
    int st_end = st_begin + P.stages_per_split;
    if (st_end > P.nstages) st_end = P.nstages;
    const int my_stages = st_end - st_begin;
    const int my_stages_pad = (my_stages + NB - 1) / NB * NB;
    const int chan_per_group = KCH / P.D2C;                  // D2C is 1, 2 or 4
    const int g_step = chan_per_group * P.cs * 4;           // bytes per channel group
    const int kp_step = KCH * P.colsp * 16;
    const int row_skip = (P.W - P.kw + 1) * pix_bytes;
    int issued = 0;
    int tap = st_begin % P.ntaps, grp = st_begin / P.ntaps;
    int tap_q = tap % P.kw;
    int tap_off = ((tap / P.kw) * P.W + tap_q) * pix_bytes;
    int g_off = grp * g_step;
    int c0 = grp * chan_per_group;  // first channel of the group
    int kp_off = (int)((((long long)d0 * P.nstages + st_begin) * KCH * P.colsp + col0) * 16);
    int q_off[KCH], q_chan[KCH];
#pragma unroll
    for (int q = 0; q < KCH; ++q) {
        q_chan[q] = q / P.D2C;
        q_off[q] = (q_chan[q] * P.cs + (q % P.D2C) * CW) * 4;
    }
    int b_const[BPW];
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
        const int c = wave * BPW + j;
        b_const[j] = ((c / (BNL / 64)) * P.colsp + (c % (BNL / 64)) * 64) * 16;
    }
    const unsigned b_voff = (unsigned)lane * 16u;

    auto issue_stage = [&](int slot) {
        const bool live = issued < my_stages;
        const unsigned stage = lds0 + slot * STAGE_BYTES;
        // input side: this lane's row, chunks 0..KCH-1 of the stage
        const bool ok = live && ((tap_ok >> tap) & 1ull) != 0;
        const unsigned voff = ok ? (unsigned)row_off : (unsigned)OOB;
        const int s_base = tap_off + g_off;
#pragma unroll
        for (int q = 0; q < KCH; ++q) {
            const bool chan_ok = c0 + q_chan[q] < P.C;  // last group may be partial
            copy_to_lds_dwords<CW>(chan_ok ? rs_in : rs_none, stage + (q * BM + 64 * wave) * 16, voff,
                            s_base + q_off[q]);
        }
        // kernel side: this wave's share of the stage's KCH x BNL chunks
#pragma unroll
        for (int j = 0; j < BPW; ++j) {
            const int c = wave * BPW + j;
            copy_to_lds_dwords<4>(rs_kp, stage + A_BYTES + c * 1024, b_voff,
                           live ? kp_off + b_const[j] : OOB);
        }
        // next stage: next tap, after the last tap the next channel group
        ++issued;
        kp_off += kp_step;
        ++tap;
        ++tap_q;
        const bool row_end = tap_q == P.kw;
        tap_q = row_end ? 0 : tap_q;
        tap_off += row_end ? row_skip : pix_bytes;
        if (tap == P.ntaps) {
            tap = 0;
            tap_q = 0;
            tap_off = 0;
            g_off += g_step;
            c0 += chan_per_group;
        }
    };

    float16v acc[TN][TM];
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

    auto compute_stage = [&](int slot) {
        const char* stage = smem + slot * STAGE_BYTES;
#pragma unroll
        for (int t = 0; t < KCH / 2; ++t) {
            // lanes 0..31 take chunk 2t, lanes 32..63 chunk 2t+1
            float4v ka[TN], ib[TM];
#pragma unroll
            for (int a = 0; a < TN; ++a)
                ka[a] = *reinterpret_cast<const float4v*>(
                    stage + A_BYTES + ((2 * t + h) * BNL + a * 32 + lr) * 16);
#pragma unroll
            for (int b = 0; b < TM; ++b)
                ib[b] = *reinterpret_cast<const float4v*>(
                    stage + ((2 * t + h) * BM + 64 * wave + b * 32 + lr) * 16);
#pragma unroll
            for (int a = 0; a < TN; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    Mma<Tag>::run(__builtin_bit_cast(chunk_t, ka[a]),
                                  __builtin_bit_cast(chunk_t, ib[b]), acc[a][b]);
        }
    };

    // ---- prologue: NB-1 stages in flight, the first one landed
    static_for<NB - 1>([&](auto S0) { issue_stage(decltype(S0)::value); });
    __builtin_amdgcn_s_waitcnt(VMCNT_KEEP);
    __syncthreads();

    // ---- main loop: copy stage s+NB-1 into the slot read in iteration s-1, contract stage s
    for (int st = 0; st < my_stages_pad; st += NB) {
        static_for<NB>([&](auto SLOT) {
            constexpr int slot = decltype(SLOT)::value;
            issue_stage((slot + NB - 1) % NB);
            compute_stage(slot);
            // this wave's copies of the next stage have landed, its reads of this stage are
            // done; after the barrier both hold for every wave
            __builtin_amdgcn_s_waitcnt(VMCNT_KEEP & 0xF0FF);
            __syncthreads();
        });
    }

    // ---- epilogue: lane (h, lr) of tile (a, b) holds in registers 4g..4g+3 the columns
    // 8g + 4h + 0..3 of the tile for output row lr of the tile
    // (partial sums of a split K loop are fp32; the reduction rounds)
    float* __restrict__ out = P.out + (long long)split * P.out_elems;
    const int caps_out = P.D0 * P.D1 * P.D3;
    const bool st4 = (P.D3 & 3) == 0;
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const long long orow = row0 + 64 * wave + b * 32 + lr;
        if (orow >= P.rows) continue;
        const long long pixel = orow / P.D1;
        const int d1 = (int)(orow % P.D1);
        long long pix_at = pixel * P.M * caps_out;
        if (P.out_mode & 1) {
            const long long n = pixel / hw;
            const int rem = (int)(pixel - n * hw);
            const int x = rem / P.Wo, y = rem - x * P.Wo;
            pix_at = P.out_base + n * P.out_sn + x * P.out_sx + y * P.out_sy;
        }
        const long long orow_off = pix_at + (long long)(d0 * P.D1 + d1) * P.D3;
#pragma unroll
        for (int a = 0; a < TN; ++a) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int j0 = col0 + a * 32 + 8 * g + 4 * h;
                if (st4) {
                    if (j0 < P.cols) {
                        const int m = j0 / P.D3, d3 = j0 - m * P.D3;
                        float4v v = {acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                                     acc[a][b][4 * g + 3]};
                        store4(out, orow_off + (long long)m * caps_out + d3, v, o16);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = j0 + u;
                        if (j < P.cols) {
                            // j / D3 by multiplication (exact while j * D3 < 2^32, which the host has checked)
                            const int m = P.d3_magic ? (int)__umulhi((unsigned)j, P.d3_magic) : j / P.D3;
                            const int d3 = j - m * P.D3;
                            store1(out, orow_off + (long long)m * caps_out + d3, acc[a][b][4 * g + u], o16);
                        }
                    }
                }
            }
        }
    }
}

template <typename Tag, int TN, int NW, int KCH, bool OUT16 = false>
hipError_t launch_kch(const Dma32Params& P, long long blocks, hipStream_t stream)
{
    constexpr int BM = 64 * NW, BNL = (32 * TN + 63) / 64 * 64;
    auto kern = igemm32_dma_kernel<Tag, TN, NW, KCH, OUT16>;
    const size_t lds_bytes = (size_t)ring_depth(KCH, TN, NW) * KCH * (BM + BNL) * 16;
    static std::atomic<unsigned long long> lds_set{0};
    hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), (int)lds_bytes, lds_set);
    if (err != hipSuccess) return err;
    kern<<<dim3((unsigned)blocks), dim3(64 * NW), lds_bytes, stream>>>(P);
    return hipGetLastError();
}

// 2-chunk stages where the column copies still divide over the waves; 16-bit output straight from
// the kernel unless a split K loop leaves fp32 partial sums for the reduction
template <typename Tag, int TN, int NW>
hipError_t launch_one(const Dma32Params& P, long long blocks, hipStream_t stream)
{
    const bool o16 = (P.out_mode >> 1) != 0 && P.nsplit == 1;
    if constexpr ((2 * ((32 * TN + 63) / 64)) % NW == 0) {
        if (P.kch == 2)
            return o16 ? launch_kch<Tag, TN, NW, 2, true>(P, blocks, stream)
                       : launch_kch<Tag, TN, NW, 2>(P, blocks, stream);
    }
    return o16 ? launch_kch<Tag, TN, NW, 4, true>(P, blocks, stream)
               : launch_kch<Tag, TN, NW, 4>(P, blocks, stream);
}

template <typename Tag, int NW>
hipError_t launch_tn(const Dma32Params& P, int tn, long long blocks, hipStream_t stream)
{
    switch (tn) {
        case 1: return launch_one<Tag, 1, NW>(P, blocks, stream);
        case 2: return launch_one<Tag, 2, NW>(P, blocks, stream);
        case 3: return launch_one<Tag, 3, NW>(P, blocks, stream);
        default: return launch_one<Tag, 4, NW>(P, blocks, stream);
    }
}

// 8-byte units: dst[pixel][c/2][d0*D1 + d1][c%2] = src[pixel][c][d0*D1 + d1]; a thread moves
// the two units of one (pixel, channel pair, row): one 16-byte store
__global__ __launch_bounds__(256) void pair_channels_kernel(const uint2* __restrict__ src,
                                                            uint4* __restrict__ dst, int C,
                                                            int rows_per_capsule, size_t pairs)
{
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= pairs) return;
    size_t r = id;
    const int row = (int)(r % rows_per_capsule); r /= rows_per_capsule;
    const int c2 = (int)(r % (C / 2));
    const size_t pixel = r / (C / 2);
    const uint2* p = src + (pixel * C + 2 * c2) * rows_per_capsule + row;
    const uint2 lo = p[0], hi = p[rows_per_capsule];
    dst[id] = uint4{lo.x, lo.y, hi.x, hi.y};
}

inline int ceil_div_ll(long long a, long long b) { return (int)((a + b - 1) / b); }

}  // namespace

// Valid floats per 16-byte chunk: 4 or 3, such that a capsule row is 1, 2 or 4 chunks (so that
// the 4 chunks of a stage never split a row); 0 if neither fits.
int igemm32_dma_chunk_width(const ConvShape& s)
{
    // 16-bit operands: capsule rows of 8, 16 or 32 halves are rows of 4, 8 or 16 "floats" as they
    // lie in memory; rows of 4 halves need an even number of channels, which a pre-pass pairs so
    // that a chunk is (c, c+1) x 4 halves
    if (s.dtype != 0) {
        if (s.D2 == 8 || s.D2 == 16 || s.D2 == 32) return 4;
        return s.D2 == 4 && s.C % 2 == 0 ? 4 : 0;
    }
    for (int cw : {4, 3}) {
        if (s.D2 % cw) continue;
        const int d2c = s.D2 / cw;
        if (d2c == 1 || d2c == 2 || d2c == 4) return cw;
    }
    return 0;
}

bool igemm32_dma_eligible(const ConvShape& s)
{
    const int cw = igemm32_dma_chunk_width(s);
    if (cw == 0) return false;
    if (s.kh * s.kw > 64) return false;                   // one mask bit per window tap
    const int es = s.dtype == 0 ? 4 : 2;
    const long long img_bytes = (long long)s.H * s.W * s.C * s.D0 * s.D1 * s.D2 * es;
    const long long hw = (long long)s.Ho * s.Wo;
    const long long pix = (256 + s.D1 - 1) / s.D1 + 1;
    const long long images_spanned = (pix + hw - 2) / hw + 1;
    const long long bias = ((long long)(s.pad > 0 ? s.pad : 0) * s.W + (s.padw() > 0 ? s.padw() : 0)) *
                           s.C * s.D0 * s.D1 * s.D2 * es;
    if (images_spanned * img_bytes + bias >= (1LL << 31)) return false;
    // (fp32 kernel: row numbers within the images a tile touches are 32-bit)
    if (s.dtype == 0 && (hw + 256) * s.D1 >= (1LL << 31)) return false;
    const Dma32Plan pl = igemm32_dma_plan(s);
    // an output view is written by the kernel itself: no partial sums over a split K loop
    if (s.out_view && (pl.P.nsplit != 1 || s.out_sn < 0 || s.out_sx < 0 || s.out_sy < 0)) return false;
    if ((long long)pl.repack_bytes >= (1LL << 31) - (1 << 24)) return false;
    return pl.blocks > 0 && pl.blocks < 0x7fffffffLL;
}

// Tile, split and padding decisions (host side, pure arithmetic).
Dma32Plan igemm32_dma_plan(const ConvShape& s)
{
    Dma32Plan pl{};
    Dma32Params& P = pl.P;
    const int cw = igemm32_dma_chunk_width(s);
    pl.cw = cw;
    pl.dtype = s.dtype;
    // 16-bit operands: in units of 4 bytes the channel-paired input is an fp32 layer with half
    // the channels and capsule rows of 4 "floats"
    const bool paired = s.dtype != 0 && s.D2 == 4;
    const int C = paired ? s.C / 2 : s.C;
    const int D2 = s.dtype == 0 ? s.D2 : paired ? 4 : s.D2 / 2;
    pl.pair_bytes = paired && !s.in_paired ? (size_t)s.in_elems() * 2 : 0;
    P.H = s.H; P.W = s.W; P.C = C; P.M = s.M; P.stride = s.stride; P.pad = s.pad;
    P.pad_w = s.padw();
    P.out_mode = (s.out_view ? 1 : 0) | (s.out16 << 1);
    P.out_base = s.out_base; P.out_sn = s.out_sn; P.out_sx = s.out_sx; P.out_sy = s.out_sy;
    P.D0 = s.D0; P.D1 = s.D1; P.D2 = D2; P.D3 = s.D3; P.Ho = s.Ho; P.Wo = s.Wo;
    P.kh = s.kh; P.kw = s.kw; P.ntaps = s.kh * s.kw;
    P.rows = s.pixels() * s.D1;
    P.out_elems = (long long)s.out_elems();
    P.pixsz = (long long)C * s.D0 * s.D1 * D2;
    P.cs = s.D0 * s.D1 * D2;
    P.cols = s.M * s.D3;
    P.D2C = cw ? D2 / cw : 1;
    const int KK = C * P.D2C;                   // chunks per row and tap
    pl.tn = P.cols <= 32 ? 1 : P.cols <= 64 ? 2 : P.cols <= 96 ? 3 : 4;
    // (fp32: columns of a tile, see igemm32_split.hip; where four column tiles pad further than
    // three, three)
    int BN = 32 * pl.tn;
    if (s.dtype == 0) {
        auto columns = [&](int tn) { return igemm32_split_tile_columns(s.D3, tn); };
        auto padded = [&](int tn) { return (P.cols + columns(tn) - 1) / columns(tn) * 32 * tn; };
        pl.tn = 1;
        while (pl.tn < 4 && P.cols > columns(pl.tn)) ++pl.tn;
        if (pl.tn == 4 && padded(3) < padded(4)) pl.tn = 3;
        BN = columns(pl.tn);
    }
    // four waves per block (256 rows) when that still fills the chip, else one (64 rows).  fp32: one
    // wave where such tiles fill the chip twice over without a split K loop, else four waves and a
    // split (64 channels of 4x4 capsules, 14x14 pixels: 98 tiles of 256 rows split 72 us, 64-row
    // tiles 80 us; 196 tiles of 256 rows split 101 us, 784 64-row tiles 87 us)
    {
        const long long cols_d0 = (long long)((P.cols + BN - 1) / BN) * s.D0;
        const long long big = (long long)ceil_div_ll(s.pixels() * s.D1, 256) * cols_d0;
        pl.nw = big >= 256 ? 4 : 1;
        if (s.dtype == 0 && (long long)ceil_div_ll(s.pixels() * s.D1, 64) * cols_d0 < 560) pl.nw = 4;
    }
    // 16-bit: chunks per stage: 2 for the four-wave tile with wide column tiles and short capsule
    // rows (4 .. 5 % faster than 4; 8-chunk stages, one workgroup per CU, 22 % slower), else 4
    // (vector capsules, whose consecutive rows are different pixels: a lane's 4 chunks are one
    // 64-byte run of memory; 11 .. 26 % faster than 2-chunk stages).  fp32: 4
    const int KCH = (s.dtype != 0 && pl.nw == 4 && pl.tn >= 3 && P.D2C <= 2 && s.D1 > 2) ? 2 : 4;
    P.kch = KCH;
    const int groups = (KK + KCH - 1) / KCH;
    pl.kqp = groups * KCH;
    P.nstages = groups * P.ntaps;
    P.col_tiles = (P.cols + BN - 1) / BN;
    P.colsp = P.col_tiles * 32 * pl.tn;
    P.row_tiles = ceil_div_ll(P.rows, 64 * pl.nw);
    const long long tiles = (long long)P.row_tiles * P.col_tiles * s.D0;
    int nsplit = 1;
    if (tiles < 256) {
        nsplit = ceil_div_ll(s.dtype == 0 ? 256 : 512, tiles);
        if (nsplit > P.nstages) nsplit = P.nstages;
        if (nsplit > 64) nsplit = 64;
    }
    P.stages_per_split = (P.nstages + nsplit - 1) / nsplit;
    if (s.dtype == 0) {  // a split begins at a whole K step
        const int per = igemm32_split_period(cw);
        P.stages_per_split = (P.stages_per_split + per - 1) / per * per;
        P.ksteps = igemm32_split_ksteps(cw, P.nstages);
    }
    P.nsplit = (P.nstages + P.stages_per_split - 1) / P.stages_per_split;
    pl.blocks = tiles * P.nsplit;
    pl.repack_bytes = s.dtype == 0 ? (size_t)s.D0 * P.ksteps * 6 * P.colsp * 16
                                   : (size_t)s.D0 * P.nstages * KCH * P.colsp * 16;
    pl.partial_bytes = P.nsplit > 1 ? (size_t)P.nsplit * P.out_elems * sizeof(float) : 0;
    P.in_bytes = (long long)s.in_elems() * (s.dtype == 0 ? 4 : 2);
    P.kp_bytes = (long long)pl.repack_bytes;
    P.d3_magic = s.D3 > 1 && (long long)s.M * s.D3 * s.D3 < (1LL << 32)
                     ? (unsigned)(((1ULL << 32) + s.D3 - 1) / s.D3)
                     : 0u;  // 0: divide
    P.xcd_span = 0;
    // (config 2: 0.90 -> 0.82 ms; with a repacked kernel far beyond the 4 MB of an L2 every
    // XCD would stream all of it per round of tiles, so large ones keep the plain order)
    if (pl.repack_bytes <= ((size_t)8 << 20)) {
        const long long unit = 8LL * s.D0 * P.col_tiles;
        const long long span = pl.blocks / unit * unit;
        if (span > 0 && span < (1LL << 31)) P.xcd_span = (int)span;
    }
    return pl;
}

namespace {

// Estimated times of an fp32 layer, us, least-squares fits over 730 random layers of 0.3 .. 8 GFLOP (most
// within 15 % of the measured time): three launches, the stages of the rounds of tiles, partial sums and the
// packed kernel written and read ...  (Fitted before the splitting left the matrix cores' pipe and the packing took a
// thread per pair: 15 random layers of up to 8 GFLOP since take 0.87 of the time, so that layers near the line may stay on
// the other kernels.)
double split_us(const Dma32Plan& pl)
{
    const double rounds = ceil((double)pl.blocks / (pl.nw == 4 ? 512 : 1024));
    const int stages = pl.P.nsplit > 1 ? pl.P.stages_per_split : pl.P.nstages;
    return 12 + (pl.P.nsplit > 1 ? 4.6 : 0) + (0.27 * pl.tn + 0.20) * stages * rounds +
           0.48e-6 * (double)pl.partial_bytes + 0.45e-6 * (double)pl.repack_bytes;
}
// ... and the kernel it would run on otherwise: the FLOPs of its tiles at the rate its input loads allow
// (16 bytes; 8 for rows of 6 floats; element by element for rows of 3)
double other_fp32_us(const ConvShape& s)
{
    const bool small = igemm_small_preferred(s);
    const long long rows = (s.pixels() * s.D1 + 63) / 64 * 64, unit = small ? 16 : 64;
    const long long cols = ((long long)s.M * s.D3 + unit - 1) / unit * unit;
    const double gflop = 2e-9 * (double)rows * (double)cols * s.D0 * s.kh * s.kw * s.C * s.D2;
    if (small) return 7.5 + gflop * (s.D2 == 3 ? 33 : s.D2 == 6 ? 28 : 14.4);
    return 12 + gflop * (s.D2 == 3 ? 21 : s.D2 == 6 ? 18 : 13.6);
}

}  // namespace

double igemm32_us(const ConvShape& s, MfmaKernel which)
{
    return which == MfmaKernel::Dma32 ? split_us(igemm32_dma_plan(s)) : other_fp32_us(s);
}

bool igemm32_dma_fills_chip(const ConvShape& s)
{
    const Dma32Plan pl = igemm32_dma_plan(s);
    return pl.nw == 4 && pl.P.nsplit == 1;
}

bool igemm32_dma_preferred(const ConvShape& s)
{
    // (most small layers leave here, before any plan is made: every rule below asks for 128 tiles of
    // 256 rows, or in fp32 for that many FLOPs, and a tile has at least 30 columns)
    const double flops = 2.0 * (double)s.out_elems() * s.kh * s.kw * s.C * s.D2;
    const double most_tiles = (double)((s.pixels() * s.D1 + 255) / 256) *
                              (double)(((long long)s.M * s.D3 + 29) / 30) * s.D0;
    if (most_tiles < 128 && !(s.dtype == 0 && flops >= 5e8)) return false;
    if (!igemm32_dma_eligible(s)) return false;
    // fp32: where its four-wave tiles fill the chip, and from 5e8 FLOPs on where it is estimated to be the
    // faster one (7.4 GFLOP of 4x4 capsules 72 against 104 us on the small-problem kernel; 3x3x3 capsules of 1.5
    // GFLOP 36 against 72; 4 images through a fully-connected layer of 12x12 capsules 70 against 20).  Of 730
    // random layers of 0.3 .. 8 GFLOP, of those taken 17 are slower than on the other kernels, by up to
    // 28 % (3 .. 10 us), 37 left to the others would gain more than 3 %; with FLOPs alone, from 5e8 (3k
    // floats) and 3e9, 82 and 56.  Layers of few columns, else on the wavefront-level path, are 1.1 .. 20 times
    // faster from 5e8 on.  Input gradients read the kernel tensor transposed, which the small-problem kernel
    // does with strides: from 5e8 and 3e9 FLOPs (5x9x6 pixels, 48 -> 8 channels of 12x12 capsules spread out
    // from stride 2: 53 against 166 us), but for those of few rows (a fully-connected layer's).
    if (s.dtype == 0) {
        const Dma32Plan pl = igemm32_dma_plan(s);
        if (pl.nw == 4 && (long long)pl.P.row_tiles * pl.P.col_tiles * s.D0 >= 256) return true;
        if (flops < 5e8) return false;
        if (few_columns(s)) return true;
        if (s.in_gradient && pl.P.rows >= 256 && flops >= (pl.cw == 3 ? 5e8 : 3e9)) return true;
        return split_us(pl) < 0.95 * other_fp32_us(s);
    }
    // 16-bit: square capsules of 8 or 16 rows belong to the 256x256-tile kernel, which is 1.12 ..
    // 1.17x faster on whole column tiles (configs 3 and 5: 0.92 against 1.03 ms, 14.2 against
    // 16.6 ms) -- unless its 256-column tiles pad the columns much further than this kernel's
    // 128-column ones (320 or 384 columns: this kernel 14 % and 7 % faster)
    if (igemm16_fast_preferred(s)) {
        const long long cols = (long long)s.M * s.D3;
        const long long pad256 = (cols + 255) / 256 * 256, pad128 = (cols + 127) / 128 * 128;
        if (pad256 * 100 < pad128 * 115) return false;
    }
    // Fewer tiles than CUs (128 .. 255 of 256 rows), and too few for the 256x256-tile kernel's rule: with
    // one-wave tiles (a split K loop where few row tiles meet many columns), from 9e9 nominal FLOPs on.  59
    // random layers of 9 .. 240 GFLOP against the any-shape kernel: 0.98 .. 2.5 times as fast, median 1.4 (14x14
    // images: 14.8 GFLOP of 4x4 capsules 51 against 60 us, of 1x8 . 8x16 capsules 42 against 54; 7.4 GFLOP of
    // 4x4 39 against 37).  The line at 128 tiles is not where the gain ends: a layer of 32 (8x8 capsules, 9.7
    // GFLOP) takes 65 us on the any-shape kernel, 50 on this one.  Square capsules of 8 and 16 rows run up to
    // 1.5 times faster still where the 256x256-tile kernel is forced (237 GFLOP of 16x16: 403 us here, 271).
    const Dma32Plan pl = igemm32_dma_plan(s);
    if (pl.nw == 4 && pl.P.nsplit == 1) return true;
    const long long tiles = (long long)ceil_div_ll(pl.P.rows, 256) * pl.P.col_tiles * s.D0;
    return tiles >= 128 && !igemm16_fast_preferred(s) &&
           flops >= 9e9;
}

hipError_t launch_igemm32_dma(const Dma32Plan& pl, hipStream_t stream)
{
    if (pl.dtype == 1)
        return pl.nw == 4 ? launch_tn<bf16_tag, 4>(pl.P, pl.tn, pl.blocks, stream)
                          : launch_tn<bf16_tag, 1>(pl.P, pl.tn, pl.blocks, stream);
    if (pl.dtype == 2)
        return pl.nw == 4 ? launch_tn<f16_tag, 4>(pl.P, pl.tn, pl.blocks, stream)
                          : launch_tn<f16_tag, 1>(pl.P, pl.tn, pl.blocks, stream);
    return launch_igemm32_split(pl, stream);
}

hipError_t launch_pair_channels(const void* src, void* dst, size_t pixels, int C,
                                int rows_per_capsule, hipStream_t stream)
{
    const size_t pairs = pixels * (size_t)(C / 2) * rows_per_capsule;  // 16 bytes each
    const size_t blocks = (pairs + 255) / 256;
    if (blocks == 0 || blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    pair_channels_kernel<<<(unsigned)blocks, 256, 0, stream>>>(
        static_cast<const uint2*>(src), static_cast<uint4*>(dst), C, rows_per_capsule, pairs);
    return hipGetLastError();
}

hipError_t launch_pair_channels(const ConvShape& s, const void* src, void* dst, hipStream_t stream)
{
    return launch_pair_channels(src, dst, (size_t)s.N * s.H * s.W, s.C, s.D0 * s.D1, stream);
}

}  // namespace capscaps
