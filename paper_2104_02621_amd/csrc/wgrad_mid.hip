// Kernel gradient of layers too small for the tiles of wgrad16.hip and wgrad32.hip (16-bit types; fp32 on the
// fp32 matrix instructions): per
// window tap one GEMM with rows (c, d2), columns (m, d3) and K (n, x, y, d1), both tensors read
// in place, whatever the channel counts.
//
// What bounds such a layer on large tiles is set-up, tiles that are mostly empty (few channels) and, for 4x4
// capsules, the two pre-passes that pair their channels.  Here the building blocks are those of
// igemm_mid.hip: copies of 64 rows x 8 K lines (1 KB) as the capsules lie in memory, operands gathered
// by the transposing LDS read on both sides (a line is one (pixel, d1), so consecutive memory is
// consecutive rows), tiles of 64 or 128 rows and columns.
//   * Rows are blocks of 64, (tap, block) in one list.  Without padding a tile's two blocks may belong to two
//     taps, so a layer of 64 rows fills 128-row tiles; with padding a tile has one tap.
//   * Every output pixel is walked; where the tap lies outside the image both sides read zeros (an
//     infinity in the gradient there must not meet a zero of the padding).
//   * The walk is done 64 pixels at a time, one per lane; a copy takes its pixel's offsets from that lane
//     (capsules of 8 and 16 rows: one pixel per copy, a lane read; of 1, 2, 4: 8, 4, 2 pixels per copy,
//     each lane fetches its own).
//   * The K loop is cut into equal ranges over workgroups; splitk_reduce adds the pieces in a fixed order.
#include <algorithm>
#include <atomic>

#include "igemm_common.h"
#include "lds_dma.h"
#include "mid_tiles.h"

namespace capscaps {
namespace {

struct WmidParams {
    const void* in;
    const void* g;
    float* out;  // dK, or partial sums [split][out_elems]
    unsigned in_bytes, g_bytes;
    int H, W, stride, pad, kw, C;
    int pix_bytes, gpix_bytes, line_in, line_g, in_sd0, g_sd0, in_sc, g_sm;  // bytes
    int rows, cols, d2_shift, d3_shift;
    int blocks_per_tap, row_blocks;  // blocks of 64 rows
    int row_tiles, col_tiles, D0, tiles, xcd_per;
    int pixels, kbs, stages_per_split, nsplit;
    FastDiv by_wo, by_ho;
    int Wo, Ho, out_sm, out_sd0;   // elements
    long long out_elems;
};

// WIDE: rows and columns come in 16-byte chunks (D2 and D3 multiples of 8, in fp32 of 4), else both are 4 (and
// D1 = 4).  fp32: a K block is 4 lines, a slot 4 columns of one, and a lane reads its column's 4 values one by one.
// (LDS holds two or three workgroups per CU.  Left to aim at four waves per SIMD the compiler waits for each K step's
// reads before it issues the next: kernel gradients of vector capsules took 1.2 times as long.)
template <typename Tag, int D1, bool WIDE, int RA, int RB, int KBS, int NST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void wgrad_mid_kernel(const WmidParams P)
{
    constexpr int A_BYTES = KBS * RA * 1024, STAGE = KBS * (RA + RB) * 1024;
    constexpr int NKB = KBS / 4, NCOPY = NKB * (RA + RB);
    constexpr int KEEP = (NST - 2) * NCOPY;
    static_assert(KEEP < 64, "vmcnt is a 6-bit counter");
    constexpr bool F32 = std::is_same_v<Tag, f32_tag>;
    constexpr int ES = F32 ? 4 : 2, LINES = F32 ? 4 : 8;  // K lines per K block
    constexpr int PPB = D1 < LINES ? LINES / D1 : 1;    // pixels per K block
    constexpr int HALVES = D1 > LINES ? D1 / LINES : 1;  // K blocks per pixel
    static_assert(HALVES <= 4, "a wave's K blocks are every fourth: always the same part of a pixel");
    // accumulators: one per K step of a stage (128x128 tiles: one), added to a second set every FLUSH stages, so
    // that chains of roundings stay short: K loops are long here
    constexpr int NACC = RA * RB == 4 ? 1 : KBS / 2, FLUSH = F32 ? 4 : RA * RB == 1 ? 32 : 16;
    extern __shared__ char smem[];

    int L = blockIdx.x;
    if (L < P.xcd_per * 8) L = (L & 7) * P.xcd_per + (L >> 3);
    const int split = L / P.tiles;
    int t = L - split * P.tiles;
    const int per_d0 = P.tiles / P.D0, d0 = t / per_d0;
    t -= d0 * per_d0;
    const int row_tile = t / P.col_tiles, col0 = (t - row_tile * P.col_tiles) * 64 * RB;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const rsrc_t rs_in = make_rsrc(P.in, P.in_bytes), rs_g = make_rsrc(P.g, P.g_bytes);

    // ---- copy side: what lane i copies of a unit.  WIDE: line (i & 7) XOR 4 in every other pair of chunks,
    // columns 8 (i >> 3) ..; else pixel i >> 5, capsule (i >> 1) & 15, lines 2 (i & 1) and the next
    const int j8 = F32 ? lane >> 2 : lane >> 3;
    const int line = F32 ? (lane & 3) ^ (j8 >> 2 & 3) : WIDE ? (lane & 7) ^ (((j8 >> 1) & 1) << 2) : (lane & 1) * 2;
    const int psub = WIDE ? (D1 < LINES ? line / D1 : 0) : lane >> 5;
    const int d1 = WIDE ? line % (D1 < LINES ? D1 : LINES) + wave % HALVES * LINES : line;
    const int first_col = F32 ? 4 * j8 : WIDE ? 8 * j8 : 4 * ((lane >> 1) & 15);
    int tap_p[RA], tap_q[RA];
    unsigned a_off[RA], b_off[RB];
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        // (blocks and rows past the last are copies of others, never stored)
        int b = row_tile * RA + i;
        b = b < P.row_blocks ? b : P.row_blocks - 1;
        const int tap = b / P.blocks_per_tap;
        int r = (b - tap * P.blocks_per_tap) * 64 + first_col;
        r = r < P.rows ? r : 0;
        tap_p[i] = tap / P.kw;
        tap_q[i] = tap - tap_p[i] * P.kw;
        a_off[i] = (unsigned)((r >> P.d2_shift) * P.in_sc + (r & ((1 << P.d2_shift) - 1)) * ES + d1 * P.line_in +
                              d0 * P.in_sd0);
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        int c = col0 + 64 * i + first_col;
        c = c < P.cols ? c : 0;
        b_off[i] = (unsigned)((c >> P.d3_shift) * P.g_sm + (c & ((1 << P.d3_shift) - 1)) * ES + d1 * P.line_g +
                              d0 * P.g_sd0);
    }

    // ---- the pixel walk: lane l holds the offsets (the input's per row block) of the l-th pixel of the next
    // 64 this wave copies
    const int first = split * P.stages_per_split, all = (P.kbs + KBS - 1) / KBS;
    const int last = first + P.stages_per_split < all ? first + P.stages_per_split : all;
    const int kb_end = last * KBS < P.kbs ? last * KBS : P.kbs;
    unsigned walk_a[RA], walk_g = OOB;
#pragma unroll
    for (int i = 0; i < RA; ++i) walk_a[i] = OOB;
    auto walk = [&](int idx) {
        const int kb = first * KBS + wave + 4 * (idx + lane / PPB);
        const int pix = kb / HALVES * PPB + lane % PPB;
        const unsigned xr = div_by((unsigned)pix, P.by_wo), y = pix - xr * P.Wo;
        const unsigned n = div_by(xr, P.by_ho), x = xr - n * P.Ho;
        const bool in_k = kb < kb_end && pix < P.pixels;
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const int h = (int)x * P.stride + tap_p[i] - P.pad, w = (int)y * P.stride + tap_q[i] - P.pad;
            const bool ok = in_k && (unsigned)h < (unsigned)P.H && (unsigned)w < (unsigned)P.W;
            walk_a[i] = ok ? ((n * P.H + (unsigned)h) * P.W + (unsigned)w) * (unsigned)P.pix_bytes : OOB;
            // (blocks of different taps: no padding, all of them inside)
            if (i == 0) walk_g = ok ? (unsigned)pix * (unsigned)P.gpix_bytes : OOB;
        }
    };
    auto of_pixel = [&](unsigned v, int l) -> unsigned {
        return PPB == 1 ? (unsigned)__builtin_amdgcn_readlane((int)v, l)
                        : (unsigned)__builtin_amdgcn_ds_bpermute((l + psub) * 4, (int)v);
    };
    auto issue = [&](int j, int slot) {
        if ((j * NKB * PPB & 63) == 0) walk(j * NKB);
#pragma unroll
        for (int u = 0; u < NKB; ++u) {
            const int kk = wave + 4 * u, l = (j * NKB + u) * PPB & 63;
            const unsigned at_g = of_pixel(walk_g, l);
#pragma unroll
            for (int i = 0; i < RA; ++i)
                copy_to_lds_dwords<4>(rs_in, (unsigned)(slot + (kk * RA + i) * 1024),
                                      a_off[i] + of_pixel(walk_a[i], l), 0);
#pragma unroll
            for (int i = 0; i < RB; ++i)
                copy_to_lds_dwords<4>(rs_g, (unsigned)(slot + A_BYTES + (kk * RB + i) * 1024), b_off[i] + at_g, 0);
        }
    };

    // ---- read side
    const int wr = wave >> 1, wc = wave & 1, half = lane >> 5, l31 = lane & 31;
    auto lane_at = [&](int c) {
        if (!F32) return transposed_at<WIDE>(lane, c);
        const int j = c / 4 + (l31 >> 2);
        return j * 64 + ((j >> 2 & 3) << 4) + (l31 & 3) * 4;
    };
    int a_rd[RA], b_rd[RB];
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        const int r = wr * 32 * RA + 32 * i;
        a_rd[i] = (half * RA + (r >> 6)) * 1024 + lane_at(r & 63);
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int c = wc * 32 * RB + 32 * i;
        b_rd[i] = A_BYTES + (half * RB + (c >> 6)) * 1024 + lane_at(c & 63);
    }
    auto read_frag = [&](int at, int rd) -> chunk_t {
        if constexpr (F32) {  // line u: address bits 4 and 5
            chunk_t v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const unsigned*>(smem + at + (rd ^ (u << 4)));
            return v;
        } else {
            return read_transposed(smem, at + rd, at + (WIDE ? rd ^ 64 : rd + 512));
        }
    };

    float16v sum[RA][RB] = {};
    int wr_slot = 0, rd_slot = 0;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
#pragma unroll
    for (int i = 0; i < NST - 1; ++i) {
        issue(i, (int)lds0 + wr_slot);
        wr_slot += STAGE;
    }
    for (int j = 0; j < last - first;) {
        float16v acc[NACC][RA][RB] = {};
        for (const int stop = j + FLUSH < last - first ? j + FLUSH : last - first; j < stop; ++j) {
            // this stage has landed, and nobody reads the slot the next copies go to any more
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(KEEP) : "memory");
            issue(j + NST - 1, (int)lds0 + wr_slot);
            wr_slot = wr_slot == (NST - 1) * STAGE ? 0 : wr_slot + STAGE;
#pragma unroll
            for (int k = 0; k < KBS / 2; ++k) {
                chunk_t fa[RA], fb[RB];
#pragma unroll
                for (int i = 0; i < RB; ++i) fb[i] = read_frag(rd_slot + k * 2 * RB * 1024, b_rd[i]);
#pragma unroll
                for (int i = 0; i < RA; ++i) fa[i] = read_frag(rd_slot + k * 2 * RA * 1024, a_rd[i]);
#pragma unroll
                for (int i = 0; i < RA; ++i)
#pragma unroll
                    for (int j2 = 0; j2 < RB; ++j2) Mma<Tag>::run(fb[j2], fa[i], acc[k % NACC][i][j2]);
            }
            rd_slot = rd_slot == (NST - 1) * STAGE ? 0 : rd_slot + STAGE;
        }
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int j2 = 0; j2 < RB; ++j2)
                sum[i][j2] += NACC == 4   ? (acc[0][i][j2] + acc[NACC / 4][i][j2]) +
                                                (acc[NACC / 2][i][j2] + acc[NACC - 1][i][j2])
                              : NACC == 2 ? acc[0][i][j2] + acc[NACC - 1][i][j2]
                                          : acc[0][i][j2];
    }
    // no copy may still be on its way into this workgroup's LDS when it ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // ---- store: a lane holds 4 consecutive columns of a row, four times per 32 columns
    float* out = P.out + (P.nsplit > 1 ? (long long)split * P.out_elems : 0);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        const int rt = wr * 32 * RA + 32 * i + l31, b = row_tile * RA + (rt >> 6);
        const int tap = b / P.blocks_per_tap, r = (b - tap * P.blocks_per_tap) * 64 + (rt & 63);
        if (b >= P.row_blocks || r >= P.rows) continue;
        const int c = r >> P.d2_shift, d2 = r & ((1 << P.d2_shift) - 1);
        const long long at = ((long long)tap * P.C + c) * ((long long)(P.cols >> P.d3_shift) * P.out_sm) +
                             (long long)d0 * P.out_sd0 + ((long long)d2 << P.d3_shift);
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int col = col0 + wc * 32 * RB + 32 * j + 8 * u + 4 * half;
                if (col >= P.cols) continue;
                const int m = col >> P.d3_shift, d3 = col & ((1 << P.d3_shift) - 1);
                const float16v& d = sum[i][j];
                const float4v v = {d[4 * u], d[4 * u + 1], d[4 * u + 2], d[4 * u + 3]};
                *reinterpret_cast<float4v*>(out + at + (long long)m * P.out_sm + d3) = v;
            }
    }
}

// Tiles, and what they take: us per stage with one, two, three workgroups on a CU, stages' worth of set-up and
// stores per workgroup, us per call.  Least-squares fits over 70 random layers of 0.003 .. 190 GFLOP, each
// with every tile and 1 .. 64 ranges (14 .. 19 % root mean square); vector capsules, whose copies gather 8 pixels,
// take 1.3 times as long.
struct Tile {
    int ra, rb, kbs, wgs;
    double us[3], extra, call;
};
constexpr Tile TILES[] = {{1, 1, 8, 3, {0.247, 0.424, 0.652}, 3.7, 3.3},
                          {1, 2, 4, 3, {0.204, 0.377, 0.444}, 8.0, 3.0},
                          {2, 1, 4, 3, {0.212, 0.347, 0.503}, 7.6, 3.0},
                          {2, 2, 4, 2, {0.303, 0.517, 0.517}, 5.7, 3.2}};

// fp32: the matrix instructions are the limit (60 layers, 6 %)
constexpr Tile TILES32[] = {{1, 1, 8, 3, {0.700, 1.196, 1.572}, 2.5, 1.5},
                            {1, 2, 4, 3, {0.668, 1.152, 1.570}, 2.5, 2.2},
                            {2, 1, 4, 3, {0.679, 1.172, 1.585}, 3.0, 1.7},
                            {2, 2, 4, 2, {1.136, 2.064, 2.064}, 1.0, 3.5}};

const Tile& tile_of(const ConvShape& s, int tile) { return s.dtype == 0 ? TILES32[tile] : TILES[tile]; }
// blocks of 64 rows per tap (see WmidParams)
int row_blocks_per_tap(const ConvShape& s, int ra)
{
    const int blocks = ceil_div((long long)s.C * s.D2, 64);
    return s.pad > 0 ? ceil_div(blocks, ra) * ra : blocks;
}
int k_blocks(const ConvShape& s) { return ceil_div(s.pixels() * s.D1, s.dtype == 0 ? 4 : 8); }

// tile and ranges: the least estimated time
MidEstimate wgrad_mid_best(const ConvShape& s, size_t room)
{
    const double out_bytes = 4.0 * (double)s.kernel_elems();
    const int kbs = k_blocks(s);
    const double slow = s.D1 <= 2 && s.dtype != 0 ? 1.3 : 1.0;
    MidEstimate best{{0, 1}, 1e30};
    for (int t = 0; t < 4; ++t) {
        const Tile& tl = tile_of(s, t);
        const long long tiles = (long long)ceil_div((long long)s.kh * s.kw * row_blocks_per_tap(s, tl.ra), tl.ra) *
                                ceil_div((long long)s.M * s.D3, 64 * tl.rb) * s.D0;
        const int all = ceil_div(kbs, tl.kbs);
        const double round = 256.0 * tl.wgs, rate = 0.95 * tl.us[tl.wgs - 1] * slow / round;
        double tile_best = 1e30;
        for (int nsplit = 1; nsplit <= 512; nsplit += nsplit < 4 ? 1 : nsplit / 4) {
            // (this and more ranges take so long at least: a workgroup's set-up, or all of them at the full chip's rate)
            const double least = std::max(tl.extra * tl.us[0], (double)tiles * (all + nsplit * tl.extra) * rate) +
                                 tl.call + (nsplit > 1 ? 3.0 + nsplit * out_bytes * 2.5e-7 : 0.0);
            if (least >= best.us) break;
            const int stages = (all + nsplit - 1) / nsplit;
            if (nsplit > 1 && (stages < 2 || (double)nsplit * out_bytes > (double)room)) break;
            const double wgs = (double)tiles * nsplit;
            const double full = (double)(long long)(wgs / round), rest = wgs - full * round;
            double us = tl.call + full * (stages + tl.extra) * tl.us[tl.wgs - 1] * slow;
            if (rest > 0) us += (stages + tl.extra) * tl.us[(int)((rest + 255) / 256) - 1] * slow;
            if (nsplit > 1) us += 3.0 + nsplit * out_bytes * 2.5e-7;
            if (us < tile_best) tile_best = us;
            if (us < best.us) best = {{t, nsplit}, us};
            // (no more ranges once they have made it slower)
            if (wgs >= 1536 || (nsplit > 2 && us > 1.1 * tile_best)) break;
        }
    }
    if (s.mid_use == 2) best.pick = asked_pick(s, best.pick, 4, out_bytes, room);
    return best;
}

struct WmidPlan {
    WmidParams P;
    int ra, rb;
    long long blocks;
};

WmidPlan wmid_plan(const ConvShape& s, MidPick pick)
{
    WmidPlan pl{};
    WmidParams& P = pl.P;
    const int es = s.dtype == 0 ? 4 : 2;
    const Tile& tl = tile_of(s, pick.tile);
    pl.ra = tl.ra;
    pl.rb = tl.rb;
    P.in_bytes = (unsigned)(s.in_elems() * es);
    P.g_bytes = (unsigned)(s.out_elems() * es);
    P.H = s.H; P.W = s.W; P.stride = s.stride; P.pad = s.pad; P.kw = s.kw; P.C = s.C; P.D0 = s.D0;
    P.line_in = s.D2 * es;
    P.line_g = s.D3 * es;
    P.in_sd0 = s.D1 * P.line_in;
    P.g_sd0 = s.D1 * P.line_g;
    P.in_sc = s.D0 * P.in_sd0;
    P.g_sm = s.D0 * P.g_sd0;
    P.pix_bytes = s.C * P.in_sc;
    P.gpix_bytes = s.M * P.g_sm;
    P.rows = s.C * s.D2;
    P.cols = s.M * s.D3;
    P.d2_shift = log2_of(s.D2);
    P.d3_shift = log2_of(s.D3);
    P.pixels = (int)s.pixels();
    P.kbs = k_blocks(s);
    P.Wo = s.Wo; P.Ho = s.Ho;
    P.by_wo = fast_div(s.Wo);
    P.by_ho = fast_div(s.Ho);
    P.out_sm = s.D0 * s.D2 * s.D3;
    P.out_sd0 = s.D2 * s.D3;
    P.out_elems = (long long)s.kernel_elems();
    P.blocks_per_tap = row_blocks_per_tap(s, pl.ra);
    P.row_blocks = s.kh * s.kw * P.blocks_per_tap;
    P.row_tiles = ceil_div(P.row_blocks, pl.ra);
    P.col_tiles = ceil_div(P.cols, 64 * pl.rb);
    P.tiles = P.row_tiles * P.col_tiles * s.D0;
    P.stages_per_split = ceil_div(ceil_div(P.kbs, tl.kbs), pick.nsplit);
    P.nsplit = ceil_div(ceil_div(P.kbs, tl.kbs), P.stages_per_split);
    pl.blocks = (long long)P.tiles * P.nsplit;
    P.xcd_per = (int)(pl.blocks / 8);
    return pl;
}

template <typename Tag, int D1, bool WIDE, int RA, int RB>
hipError_t launch_tile(const WmidPlan& pl, hipStream_t stream)
{
    constexpr int KBS = RA * RB == 1 ? 8 : 4, NST = RA * RB == 1 ? 3 : 4;
    constexpr int lds = NST * KBS * (RA + RB) * 1024;
    auto kern = wgrad_mid_kernel<Tag, D1, WIDE, RA, RB, KBS, NST>;
    static std::atomic<unsigned long long> lds_set{0};
    const hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), lds, lds_set);
    if (err != hipSuccess) return err;
    kern<<<dim3((unsigned)pl.blocks), dim3(256), lds, stream>>>(pl.P);
    return hipGetLastError();
}
template <typename Tag, int D1, bool WIDE>
hipError_t launch_mode(const WmidPlan& pl, hipStream_t stream)
{
    if (pl.ra == 2) return pl.rb == 2 ? launch_tile<Tag, D1, WIDE, 2, 2>(pl, stream)
                                      : launch_tile<Tag, D1, WIDE, 2, 1>(pl, stream);
    return pl.rb == 2 ? launch_tile<Tag, D1, WIDE, 1, 2>(pl, stream)
                      : launch_tile<Tag, D1, WIDE, 1, 1>(pl, stream);
}
template <typename Tag>
hipError_t launch_tag(const WmidPlan& pl, const ConvShape& s, hipStream_t stream)
{
    if constexpr (!std::is_same_v<Tag, f32_tag>)
        if (s.D2 == 4) return launch_mode<Tag, 4, false>(pl, stream);
    switch (s.D1) {
        case 1: return launch_mode<Tag, 1, true>(pl, stream);
        case 2: return launch_mode<Tag, 2, true>(pl, stream);
        case 4: return launch_mode<Tag, 4, true>(pl, stream);
        case 8: return launch_mode<Tag, 8, true>(pl, stream);
        default: return launch_mode<Tag, 16, true>(pl, stream);
    }
}

}  // namespace

bool wgrad_mid_eligible(const ConvShape& s)
{
    if (!s.plain() || s.out16 != 0 || s.mid_use == 1) return false;
    const size_t es = s.dtype == 0 ? 4 : 2;
    if (s.dtype == 0) {
        if (s.D2 < 4 || s.D3 < 4 || !pow2(s.D2) || !pow2(s.D3) || !pow2(s.D1) || s.D1 > 16) return false;
    } else if (s.D2 == 4 || s.D3 == 4) {
        if (s.D1 != 4 || s.D2 != 4 || s.D3 != 4) return false;
    } else if (s.D2 % 8 != 0 || s.D3 % 8 != 0 || !pow2(s.D2) || !pow2(s.D3) ||
               !(s.D1 == 1 || s.D1 == 2 || s.D1 == 4 || s.D1 == 8 || s.D1 == 16)) {
        return false;
    }
    // 32-bit offsets below the out-of-range mark, also those of the pixels a K loop's end runs past
    const size_t gpix = (size_t)s.M * s.D0 * s.D1 * s.D3 * es;
    if (s.in_elems() * es >= MAX_TENSOR_BYTES || s.out_elems() * es + 512 * gpix >= MAX_TENSOR_BYTES)
        return false;
    if (s.H > (1 << 14) || s.W > (1 << 14) || s.kh > (1 << 12) || s.kw > (1 << 12) || s.pad > (1 << 14) ||
        s.stride > (1 << 14))
        return false;
    if (s.pixels() * s.D1 >= (1LL << 29) || (long long)s.C * s.D2 >= (1LL << 24) ||
        (long long)s.M * s.D3 >= (1LL << 24))
        return false;
    const long long blocks = (long long)s.kh * s.kw * ceil_div((long long)s.C * s.D2, 64);
    return blocks * ceil_div((long long)s.M * s.D3, 64) * s.D0 < (1LL << 24);
}

namespace {
// part of the output pixels that a window tap reaches, on average, in one dimension
double reached(int extent, int out, int k, int stride, int pad)
{
    if (pad == 0) return 1.0;
    long long n = 0;
    for (int t = 0; t < k; ++t) {
        const int lo = t < pad ? (pad - t + stride - 1) / stride : 0, top = extent - 1 + pad - t;
        const int hi = top < 0 ? -1 : top / stride < out ? top / stride : out - 1;
        if (hi >= lo) n += hi - lo + 1;
    }
    return (double)n / ((double)out * k);
}
}  // namespace

// Against wgrad16_kernel, which walks only the pixels that a tap reaches (estimated: 21 us and its 256 x 256 tiles' FLOPs at
// 1.23 PFLOP/s, 27 % root mean square), where this one takes at most 0.8 of the 21 us and 0.66 of the FLOPs' part, with 0.2 us per
// MB beyond the 60 that the caches hold between two taps: of 1667 random layers 1417 leave, none slower by more than 3 %, 0.44 times the
// time on average.  (By 0.8 of both and all pixels: 3 x 3, 15 -> 3 channels of 16x16, 0.5 GB, 571 -> 658 us; 6 x 6, 28 -> 5 channels
// of 8x8 on 6x6 images with padding 3, 52 -> 73; 6 x 6, 48 -> 8 channels of 1x8 . 8x16, 231 -> 334.)  Against the kernel
// gradient as a convolution always.
MidPick wgrad_mid_choice(const ConvShape& s, size_t room)
{
    if (!wgrad_mid_eligible(s)) return {};
    if (s.mid_use == 2) return wgrad_mid_best(s, room).pick;
    const bool other = s.dtype == 0 ? wgrad32_eligible(s) : wgrad16_eligible(s);
    // fp32: where estimated 15 % faster than wgrad32_kernel (47 random layers: the 22 that leave it take 0.37 .. 0.97
    // of its time)
    // and at least 64 K values (shorter sums have fewer roundings there: 3e-8 against 5e-8)
    if (other && s.dtype == 0 && s.pixels() * s.D1 < 64) return {};
    const MidEstimate e = wgrad_mid_best(s, room);
    if (!other) return e.pick;
    if (s.dtype == 0) return e.us < 0.85 * wgrad32_us(s) ? e.pick : MidPick{};
    const int rows = s.C * s.D2, cols = s.M * s.D3, nt = rows > 128 ? 1 : rows > 64 ? 2 : 4;
    const double gflop = 2e-9 * (double)(s.pixels() * s.D1) * ceil_div(s.kh * s.kw, nt) * s.D0 *
                         (256.0 * ceil_div(rows, 256)) * (256.0 * ceil_div(cols, 256));
    const double part = reached(s.H, s.Ho, s.kh, s.stride, s.pad) * reached(s.W, s.Wo, s.kw, s.stride, s.pad);
    const double mb = 2e-6 * (double)(s.in_elems() + s.out_elems());
    return e.us + 0.2 * std::max(mb - 60.0, 0.0) < 0.8 * 21.0 + 0.66 / 1.23 * gflop * part ? e.pick : MidPick{};
}

hipError_t launch_wgrad_mid(const ConvShape& s, MidPick pick, const void* input, const void* dout, float* dkernel,
                            void* workspace, hipStream_t stream)
{
    WmidPlan pl = wmid_plan(s, pick);
    pl.P.in = input;
    pl.P.g = dout;
    float* partial = static_cast<float*>(workspace);
    pl.P.out = pl.P.nsplit > 1 ? partial : dkernel;
    const hipError_t err = s.dtype == 0   ? launch_tag<f32_tag>(pl, s, stream)
                           : s.dtype == 1 ? launch_tag<bf16_tag>(pl, s, stream)
                                          : launch_tag<f16_tag>(pl, s, stream);
    if (err != hipSuccess || pl.P.nsplit == 1) return err;
    return launch_splitk_reduce(partial, dkernel, pl.P.out_elems, pl.P.nsplit, stream);
}

}  // namespace capscaps
