// Capsule convolution for layers too small for the 256-row tiles (16-bit forward pass and input gradient;
// fp32 input gradient on the fp32 matrix instructions): one launch, kernel tensor read in place, small tiles, direct-to-LDS copies.
//
// What bounds such a layer is not the matrix cores but everything around them: the launch of a
// repack pass, operands staged through registers, a reduction launch, and a K loop whose every
// stage waits for memory.  So: both operands are copied global -> LDS as they lie in memory, three
// stages ahead, in units of 1 KB = 64 rows (or columns) x 8 K values, one wave instruction each, and
// the layout a matrix instruction wants (8 consecutive K values per lane) is made by the read:
//   * rows whose K values are contiguous (the input; the kernel tensor in the input gradient):
//       capsule rows of 8k elements: 16-byte slots [K block][row], one ds_read_b128;
//       rows of 4: a slot is two rows x 4 values, a K block two channels, two ds_read_b64;
//   * columns contiguous (the kernel tensor [c][m][d2][d3] in the forward pass): the transposing
//       read ds_read_b64_tr_b16 (of a 16-lane group, lane 4a + b supplies the address of 4 columns
//       of K line a, lane i receives column i's values of the four lines), two per operand.  Slots
//       of 8 columns x 1 line, [K block][column chunk][line], the line of every other pair of
//       chunks XORed with 4 so that a half-wave's reads touch every bank once; for 4-element
//       columns a slot is 2 lines x 4 columns and the order of memory is conflict-free as it is.
// fp32 (input gradients only: its forward pass is not faster here than on igemm_small.hip's narrower tiles):
// a K block is 4 values, so rows of 4k floats are the rows of 8k halves above, byte for byte, and one
// 16-byte read feeds four matrix instructions (as in Mma<f32_tag>).
// The K blocks of a stage are a flat sequence (tap, channel block): short channel extents pad
// nothing.  A wave copies the K blocks w, w + 4 .. of a stage: one (tap, channel) walk per block in
// scalar registers, one address and range test per row in the lanes.  Out-of-range offsets read as
// zeros (padding taps, missing rows and columns, the K tail).
// The input gradient of a strided layer is stride^2 convolutions on interleaved pixels ("phases");
// all of them run in the one launch.
#include <algorithm>
#include <atomic>

#include "igemm_common.h"
#include "lds_dma.h"
#include "mid_tiles.h"

namespace capscaps {
namespace {

constexpr int MAX_PHASES = 16;
constexpr int MAX_EXTENT = 4096;  // of images, windows, paddings: the walk packs tap positions into 13 bits

struct MidPhase {
    int Ho, Wo, kw, pad_h, pad_w;
    int kbs;          // K blocks: taps * blocks per tap
    int rows;         // N * Ho * Wo * D1
    int tile0;        // first tile of the phase
    int stages_per_split;
    int kw_magic;     // ceil(2^32 / kw), 0 for kw = 1
    FastDiv by_wo, by_ho;
    int k_base;       // bytes
    long long out_base;
};
struct MidCommon {
    const void* in;
    const void* kernel;
    float* out;  // final output, or partial sums [split][out_elems]
    unsigned in_bytes, k_bytes;
    int H, W, stride, D1, C;
    int pix_bytes, d1_bytes, in_sd0;  // input: bytes per pixel, per capsule row, per leading index
    int in_kb, in_blk;                // ... per channel step of a K block, per 8 values of a row
    int kpt, kq;                      // K blocks per tap, padded to whole groups, and as they are
    unsigned kpt_magic;
    int kb_shift, kb_mask;            // K blocks per channel: 1 << kb_shift
    int k_sp, k_sq, k_kb, k_blk, k_sd0, k_sm, k_col, k_c2;  // kernel tensor, bytes
    int dc_shift;                     // log2 of the columns per output capsule row
    int cols, col_tiles, D0, tiles, nsplit, nphase, xcd_per;
    int skip_taps;                    // see sum_inside
    FastDiv by_d1;
    long long out_sn, out_sx, out_sy, out_elems;  // elements
    int out_sm, out_sd0;
};
// (a forward pass has one phase: the launch of a small one takes 0.3 us less with 0.3 KB of arguments than with 1.4)
template <int PHASES>
struct MidParams : MidCommon {
    MidPhase ph[PHASES];
};

// One copy instruction: 64 slots of 16 bytes = 64 / G rows x G K blocks, so that neighbouring lanes read
// neighbouring memory whatever the capsule shape.  Slot i holds, for
//   WIDE (capsule rows of 8k elements): row i / G, K block i % G;
//   else (rows of 4; a K block is two channels, G = 2): of four rows at a time, rows 2 (i & 1) and
//   2 (i & 1) + 1 of channel (i >> 1) & 3
// with the K block (channel) XORed by a function of the row that spreads the reads over the banks.
template <bool WIDE, int G>
__device__ __forceinline__ int slot_row(int i) { return WIDE ? i / G : 4 * (i >> 3) + 2 * (i & 1); }
template <bool WIDE, int G>
__device__ __forceinline__ int row_swizzle(int r)
{
    return !WIDE ? (r >> 2) & 3 : G == 2 ? (r >> 2) & 1 : G == 4 ? (r >> 1) & 3 : 0;
}
template <bool WIDE, int G>
__device__ __forceinline__ int slot_k(int i)  // K block of the group, or channel of the group
{
    return (WIDE ? i % G : (i >> 1) & 3) ^ row_swizzle<WIDE, G>(slot_row<WIDE, G>(i));
}
// byte of row r's values of K block kb (their first half, for rows of 4) inside a region of R * 64 rows
template <bool WIDE, int G, int R>
__device__ __forceinline__ int region_at(int r, int kb)
{
    const int g = kb % G, group = kb / G * (R * G * 1024);
    if (WIDE) return group + r * (G * 16) + ((g ^ row_swizzle<WIDE, G>(r)) << 4);
    return group + (r >> 2) * 128 + (((2 * g) ^ row_swizzle<WIDE, G>(r)) << 5) + (r & 3) * 8;
}

template <typename Tag>
__device__ __forceinline__ float value_at(const void* base, long long byte)
{
    const char* at = static_cast<const char*>(base) + byte;
    if constexpr (std::is_same_v<Tag, f32_tag>) return *reinterpret_cast<const float*>(at);
    else if constexpr (std::is_same_v<Tag, f16_tag>) return (float)*reinterpret_cast<const _Float16*>(at);
    else return __builtin_bit_cast(float, (unsigned)*reinterpret_cast<const unsigned short*>(at) << 16);
}
// One element of an input gradient (image n, window corner h, w, capsule row d1, column m, dc) as a plain sum
// over the taps inside the image.  The matrix instructions multiply the zeros outside it by the kernel tensor's values, which
// an infinite or NaN one there turns into a NaN.  (64 -> 64 channels of bf16 8x8, N = 4, 28x28, a 1x5 window: 132 us, with one
// infinite weight 0.32 ms, with nothing but NaNs 0.41; gather kernel 16.5 ms.)
template <typename Tag>
__device__ __forceinline__ float sum_inside(const MidCommon& P, const MidPhase& F, int n, int h, int w, int d0, int d1, int m, int dc)
{
    constexpr int ES = sizeof(typename Tag::elem);
    const int kh = F.kw > 0 ? F.kbs / (P.kpt * F.kw) : 0, row = P.d1_bytes / ES;
    float acc = 0.f;
    for (int p = 0; p < kh; ++p) {
        if ((unsigned)(h + p) >= (unsigned)P.H) continue;
        for (int q = 0; q < F.kw; ++q) {
            if ((unsigned)(w + q) >= (unsigned)P.W) continue;
            long long a = (((long long)n * P.H + h + p) * P.W + w + q) * P.pix_bytes + (long long)d0 * P.in_sd0 +
                          (long long)d1 * P.d1_bytes;
            long long b = F.k_base + (long long)p * P.k_sp + (long long)q * P.k_sq + (long long)d0 * P.k_sd0 +
                          (long long)m * P.k_sm + (long long)dc * P.k_col;
            for (int c = 0; c < P.C; ++c) {
                for (int e = 0; e < row; ++e)
                    acc = fmaf(value_at<Tag>(P.in, a + e * ES), value_at<Tag>(P.kernel, b + e * ES), acc);
                if (acc != acc) return acc;  // (a NaN stays one)
                a += (long long)P.D0 * P.in_sd0;
                b += P.k_c2;
            }
        }
    }
    return acc;
}

// KT: the kernel tensor has its columns contiguous (transposing read), else its K values.  Tile:
// 64*RA rows x 64*RB columns, four waves over 4 / WC rows x WC columns of them (WC = 1: 32 columns
// only); KBS K blocks (of 8) per stage, NST stages in the ring.
template <typename Tag, bool WIDE, int G, bool KT, bool OUT16, int RA, int RB, int WC, int KBS, int NST>
__global__ __launch_bounds__(256, 2) void igemm_mid_kernel(const MidParams<KT ? 1 : MAX_PHASES> P)
{
    constexpr int A_BYTES = KBS * RA * 1024, STAGE = KBS * (RA + RB) * 1024;
    constexpr int NKB = KBS / 4, NCOPY = NKB * (RA + RB);
    constexpr int TM = RA * WC / 2, TN = WC == 1 ? 1 : RB;  // 32 x 32 tiles of a wave
    constexpr bool F32 = std::is_same_v<Tag, f32_tag>;
    constexpr int BN = 32 * TN * WC;
    constexpr int KEEP = (NST - 2) * NCOPY;  // copies that may be in flight at a stage's barrier
    static_assert(KEEP < 64 && KBS % 4 == 0, "vmcnt is a 6-bit counter");
    extern __shared__ char smem[];

    // ---- which tile: columns fastest, then rows (of all phases), leading index, K split; every
    // XCD takes a contiguous range of them
    int L = blockIdx.x;
    if (L < P.xcd_per * 8) L = (L & 7) * P.xcd_per + (L >> 3);
    const int split = L / P.tiles;
    int t = L - split * P.tiles;
    const int per_d0 = P.tiles / P.D0, d0 = t / per_d0;
    t -= d0 * per_d0;
    const int row_tile_all = t / P.col_tiles, col_tile = t - row_tile_all * P.col_tiles;
    int phase = 0;
    if constexpr (!KT)
        while (phase + 1 < P.nphase && row_tile_all >= P.ph[phase + 1].tile0) ++phase;
    const MidPhase& F = P.ph[phase];
    const int row0 = (row_tile_all - F.tile0) * 64 * RA, col0 = col_tile * BN;
    const int Ho = F.Ho, Wo = F.Wo, kw = F.kw, rows = F.rows, kbs = F.kbs;
    const FastDiv by_wo = F.by_wo, by_ho = F.by_ho;
    const unsigned kw_magic = F.kw_magic, kw_one = kw == 1 ? ~0u : 0u;
    const unsigned kpt_magic = P.kpt_magic, kpt_one = P.kpt == 1 ? ~0u : 0u;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const rsrc_t rs_in = make_rsrc(P.in, P.in_bytes), rs_k = make_rsrc(P.kernel, P.k_bytes);

    // ---- copy side.  A wave copies K blocks w, w + 4 .. of a stage; of a group of G blocks that is rows
    // sub * 64 RA / G .. of the tile, all blocks
    const int sub = wave % G;
    const int ga = slot_k<WIDE, G>(lane);  // this lane's K block (channel) of the group
    int h0[RA], w0[RA];
    unsigned a_off[RA], b_off[RB];
    const unsigned a_k = WIDE ? (ga & P.kb_mask) * 16 + (ga >> P.kb_shift) * P.in_kb : ga * (P.in_kb >> 1);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        const int r = row0 + (sub * RA + i) * (64 / G) + slot_row<WIDE, G>(lane);
        const unsigned pix = div_by((unsigned)r, P.by_d1), d1 = r - pix * P.D1;
        const unsigned xr = div_by(pix, by_wo), y = pix - xr * Wo;
        const unsigned n = div_by(xr, by_ho), x = xr - n * Ho;
        h0[i] = r < rows ? (int)x * P.stride - F.pad_h : -(1 << 30);
        w0[i] = (int)y * P.stride - F.pad_w;
        a_off[i] = ((n * P.H + x * P.stride - F.pad_h) * P.W + (unsigned)w0[i]) * (unsigned)P.pix_bytes +
                   d1 * P.d1_bytes + d0 * P.in_sd0 + a_k;
    }
    const int c2 = KT ? lane >> 5 : ga;  // rows of 4: this lane's kernel channel
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        int col;
        unsigned extra;
        if (KT && WIDE) {
            const int j = lane >> 3;
            col = col0 + 64 * i + 8 * j;
            extra = ((lane & 7) ^ (((j >> 1) & 1) << 2)) * P.k_col;  // the line
        } else if (KT) {
            col = col0 + 64 * i + 4 * ((lane >> 1) & 15);
            extra = (lane & 1) * 16 + c2 * P.k_c2;
        } else {
            col = col0 + (sub * RB + i) * (64 / G) + slot_row<WIDE, G>(lane);
            extra = WIDE ? (ga & P.kb_mask) * P.k_blk + (ga >> P.kb_shift) * P.k_kb : c2 * P.k_c2;
        }
        const int m = col >> P.dc_shift, dc = col & ((1 << P.dc_shift) - 1);
        b_off[i] = col < P.cols && col < col0 + BN
                       ? (unsigned)(m * P.k_sm + dc * (KT ? 2 : P.k_col)) + extra
                       : OOB;
    }
    const unsigned b_base = (unsigned)(F.k_base + d0 * P.k_sd0);

    // ---- the walk over taps and channels, 64 of this wave's K blocks at a time: lane j holds the offsets
    // of the j-th, the copies read them out (a chain of scalar multiplications per stage took as
    // long as the stage's matrix instructions)
    const int first = split * F.stages_per_split, all = (kbs + KBS - 1) / KBS;
    const int last = first + F.stages_per_split < all ? first + F.stages_per_split : all;
    int walk_a = 0, walk_b = 0;
    unsigned walk_p = 0;
    auto walk = [&](int idx) {
        const int kb = first * KBS + wave + 4 * (idx + lane);
        const int tap = (int)(__umulhi((unsigned)kb, kpt_magic) + ((unsigned)kb & kpt_one));
        const int q = kb - tap * P.kpt, qa = q - sub;  // K block of the tap, and its group's first
        const int p = (int)(__umulhi((unsigned)tap, kw_magic) + ((unsigned)tap & kw_one));
        const int pw = tap - p * kw, qb = KT ? q : qa;
        const bool in_k = kb < kbs && kb < last * KBS;
        walk_a = (p * P.W + pw) * P.pix_bytes + (qa >> P.kb_shift) * P.in_kb + (qa & P.kb_mask) * P.in_blk;
        // (what lies past the tap's last K block, as its blocks are padded to whole groups, is out of range)
        walk_b = in_k && (!KT || G == 1 || q < P.kq)
                     ? (int)b_base + p * P.k_sp + pw * P.k_sq + (qb >> P.kb_shift) * P.k_kb +
                           (qb & P.kb_mask) * P.k_blk
                     : 0x7ffffff0;
        const int left = WIDE ? P.kq - qa : P.C - 2 * qa;  // K blocks (channels) of the tap from the group's first on
        walk_p = in_k ? (unsigned)(p | pw << 13 | (left < 7 ? left : 7) << 26) : MAX_EXTENT;
    };

    // ---- copies of stage first + j into the ring slot at byte `slot`
    auto issue = [&](int j, int slot) {
        if ((j * NKB & 63) == 0) walk(j * NKB);
#pragma unroll
        for (int u = 0; u < NKB; ++u) {
            const int kk = wave + 4 * u, l = (j * NKB + u) & 63;
            const int so_a = __builtin_amdgcn_readlane(walk_a, l), so_b = __builtin_amdgcn_readlane(walk_b, l);
            const unsigned pk = (unsigned)__builtin_amdgcn_readlane((int)walk_p, l);
            const int p = (int)(pk & 0x1fffu), pw = (int)(pk >> 13 & 0x1fffu), left = (int)(pk >> 26);
            const bool a_ok = (WIDE && G == 1) || ga < left;
            const bool b_ok = WIDE ? KT || a_ok : c2 + (KT ? 2 * sub : 0) < left;
            const unsigned dst = (unsigned)(slot + kk * RA * 1024);
#pragma unroll
            for (int i = 0; i < RA; ++i) {
                const bool ok = (unsigned)(h0[i] + p) < (unsigned)P.H &&
                                (unsigned)(w0[i] + pw) < (unsigned)P.W && a_ok;
                copy_to_lds_dwords<4>(rs_in, dst + i * 1024, ok ? a_off[i] + (unsigned)so_a : OOB, 0);
            }
#pragma unroll
            for (int i = 0; i < RB; ++i)
                copy_to_lds_dwords<4>(rs_k, (unsigned)(slot + A_BYTES + (kk * RB + i) * 1024),
                                      b_ok ? b_off[i] : OOB, so_b);
        }
    };

    // ---- read side: this lane's byte offsets inside a stage (K blocks 0 and 1, or 2 and 3)
    const int wr = wave / WC, wc = wave % WC, half = lane >> 5, l31 = lane & 31;
    const int arow = wr * 32 * TM + l31;  // + 32 * tm
    constexpr int ALT = G == 4 ? 2 : 1;   // (groups of four: the odd steps' blocks are the third and fourth)
    int a_rd[ALT][TM], b_rd[ALT][TN];
#pragma unroll
    for (int o = 0; o < ALT; ++o) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a_rd[o][i] = region_at<WIDE, G, RA>(arow + 32 * i, 2 * o + half);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int cb = wc * 32 * TN + 32 * i;  // first column of the fragment
            if (KT) {
                b_rd[o][i] = A_BYTES + ((2 * o + half) * RB + (cb >> 6)) * 1024 + transposed_at<WIDE>(lane, cb & 63);
            } else {
                b_rd[o][i] = A_BYTES + region_at<WIDE, G, RB>(cb + l31, 2 * o + half);
            }
        }
    }
    auto read_plain = [&](int at, int at2) -> chunk_t {
        if (WIDE) return *reinterpret_cast<const chunk_t*>(smem + at);
        struct { uint2 lo, hi; } v;
        v.lo = *reinterpret_cast<const uint2*>(smem + at);
        v.hi = *reinterpret_cast<const uint2*>(smem + at2);
        return __builtin_bit_cast(chunk_t, v);
    };
    // one accumulator per K step of a stage: shorter chains of roundings (with one, results of small
    // layers were up to 2.2 times as far from exact sums as the small-problem kernel's, whose waves share
    // the K loop), and matrix instructions that do not wait for each other
    constexpr int NACC = KBS / 2;
    // fp32 adds them, in pairs, to another set every FLUSH stages (an instruction takes only two K values there)
    constexpr int FLUSH = 4;
    float16v acc[NACC][TM][TN] = {}, sum[F32 ? TM : 1][TN] = {};
    int wr_slot = 0, rd_slot = 0;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
#pragma unroll
    for (int i = 0; i < NST - 1; ++i) {
        issue(i, (int)lds0 + wr_slot);
        wr_slot += STAGE;
    }
    for (int j = 0; j < last - first; ++j) {
        // this stage has landed, and nobody reads the slot the next copies go to any more
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(KEEP) : "memory");
        issue(j + NST - 1, (int)lds0 + wr_slot);
        wr_slot = wr_slot == (NST - 1) * STAGE ? 0 : wr_slot + STAGE;
#pragma unroll
        for (int k = 0; k < KBS / 2; ++k) {
            const int o = ALT == 2 ? k & 1 : 0, ka = (k - o) * 2 * RA * 1024, kb = (k - o) * 2 * RB * 1024;
            chunk_t fa[TM], fb[TN];
            // (second half of the 8 K values: the other four lines, address bit 6; the second channel,
            // bit 5 or, in the transposed layout, bit 9)
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const int at = rd_slot + kb + b_rd[o][i];
                if constexpr (KT)
                    fb[i] = read_transposed(smem, at, WIDE ? rd_slot + kb + (b_rd[o][i] ^ 64) : at + 512);
                else
                    fb[i] = read_plain(at, rd_slot + kb + (b_rd[o][i] ^ 32));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = read_plain(rd_slot + ka + a_rd[o][i], rd_slot + ka + (a_rd[o][i] ^ 32));
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) Mma<Tag>::run(fb[j], fa[i], acc[k][i][j]);
        }
        if constexpr (F32)
            if (j % FLUSH == FLUSH - 1) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        sum[i][b] += NACC == 4 ? (acc[0][i][b] + acc[1][i][b]) +
                                                     (acc[NACC - 2][i][b] + acc[NACC - 1][i][b])
                                               : acc[0][i][b] + acc[NACC - 1][i][b];
#pragma unroll
                        for (int a = 0; a < NACC; ++a) acc[a][i][b] = float16v{};
                    }
            }
        rd_slot = rd_slot == (NST - 1) * STAGE ? 0 : rd_slot + STAGE;
    }
    // no copy may still be on its way into this workgroup's LDS when it ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

#pragma unroll
    for (int w = NACC / 2; w > 0; w /= 2)
#pragma unroll
        for (int a = 0; a < w; ++a)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[a][i][j] += acc[a + w][i][j];

    if constexpr (F32) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[0][i][j] += sum[i][j];
    }

    // ---- store: a lane holds 4 consecutive columns of a row, four times per 32 columns
    float* out = P.out + (P.nsplit > 1 ? (long long)split * P.out_elems : 0);
    constexpr int KIND = OUT16 ? (std::is_same_v<Tag, f16_tag> ? 2 : 1) : 0;
    float nan = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = row0 + arow + 32 * i;
        if (r >= rows) continue;
        const unsigned pix = div_by((unsigned)r, P.by_d1), d1 = r - pix * P.D1;
        const unsigned xr = div_by(pix, by_wo), y = pix - xr * Wo;
        const unsigned n = div_by(xr, by_ho), x = xr - n * Ho;
        const long long at = F.out_base + n * P.out_sn + x * P.out_sx + y * P.out_sy +
                             (long long)(d0 * P.out_sd0) + ((long long)d1 << P.dc_shift);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int col = col0 + wc * 32 * TN + 32 * j + 8 * u + 4 * half;
                if (col >= P.cols) continue;
                const int m = col >> P.dc_shift, dc = col & ((1 << P.dc_shift) - 1);
                const float16v& d = acc[0][i][j];
                const float4v v = {d[4 * u], d[4 * u + 1], d[4 * u + 2], d[4 * u + 3]};
                store4(out, at + (long long)m * P.out_sm + dc, v, KIND);
                if constexpr (!KT)
#pragma unroll
                    for (int k = 0; k < 4; ++k) nan = fmaf(v[k], 0.f, nan);  // NaN from an infinity or a NaN
            }
    }
    // NaNs of a layer whose out-of-image taps must not count (unsplit K loops only): this lane's once more, one by one
    if constexpr (!KT)
        if (P.skip_taps && nan != 0.f)
#pragma unroll 1
            for (int t = 0; t < TM * TN * 4; ++t) {
                const int r = row0 + arow + 32 * (t / (TN * 4));
                const int col = col0 + wc * 32 * TN + 8 * (t % (TN * 4)) + 4 * half;
                if (r >= rows || col >= P.cols) continue;
                const unsigned pix = div_by((unsigned)r, P.by_d1), d1 = r - pix * P.D1;
                const unsigned xr = div_by(pix, by_wo), y = pix - xr * Wo;
                const unsigned n = div_by(xr, by_ho), x = xr - n * Ho;
                const int m = col >> P.dc_shift, dc = col & ((1 << P.dc_shift) - 1);
                const long long at = F.out_base + n * P.out_sn + x * P.out_sx + y * P.out_sy +
                                     (long long)(d0 * P.out_sd0) + ((long long)d1 << P.dc_shift) +
                                     (long long)m * P.out_sm + dc;
#pragma unroll 1
                for (int k = 0; k < 4; ++k) {
                    const float got = OUT16 ? value_at<Tag>(out, (at + k) * 2) : out[at + k];
                    if (got == got) continue;
                    store1(out, at + k, sum_inside<Tag>(P, F, (int)n, (int)x * P.stride - F.pad_h,
                                                        (int)y * P.stride - F.pad_w, d0, (int)d1, m, dc + k), KIND);
                }
            }
}

struct Strides {
    long long sp, sq, sc, sm, sd0, sd2, sd3;
};
Strides kernel_strides(const ConvShape& s)
{
    if (s.kernel_view) return {s.k_sp, s.k_sq, s.k_sc, s.k_sm, s.k_sd0, s.k_sd2, s.k_sd3};
    Strides k;
    k.sd3 = 1;
    k.sd2 = s.D3;
    k.sd0 = (long long)s.D2 * s.D3;
    k.sm = k.sd0 * s.D0;
    k.sc = k.sm * s.M;
    k.sq = k.sc * s.C;
    k.sp = k.sq * s.kw;
    return k;
}

struct MidPlan {
    MidParams<MAX_PHASES> P;
    bool wide, kt, out16;
    int ra, rb, wc, g;
    long long blocks;
};

int elem_size(const ConvShape& s) { return s.dtype == 0 ? 4 : 2; }

// K blocks per copy: rows of 32 bytes and more: both halves of 32; capsules of one or two rows: 64
// bytes of a pixel
int mid_group(const ConvShape& s)
{
    const int row = s.D2 * elem_size(s) / 2;
    if (row % 8 != 0) return 2;
    return s.D1 <= 2 ? 4 : row >= 16 ? 2 : 1;
}
// K blocks of a tap, as they are and padded to whole copies
int k_blocks(const ConvShape& s)
{
    const int row = s.D2 * elem_size(s) / 2;
    return row % 8 == 0 ? s.C << log2_of(row / 8) : (s.C + 1) / 2;
}
int padded_k_blocks(const ConvShape& s)
{
    const int g = mid_group(s);
    return (k_blocks(s) + g - 1) / g * g;
}

// Tiles, and what they take: us per stage with one, two, three workgroups on a CU, stages' worth of
// set-up and stores per workgroup, us per call.  Least-squares fits over 180 random layers of 0.003 .. 200
// GFLOP, each timed with every tile and 1 .. 8 pieces of the K loop (2500 times; 17 % root mean square).
// One workgroup's stage is a chain of waits; of several on a CU the 64 bytes per cycle of the L1 and, for
// 64x64 tiles, the LDS reads are the limit.
struct Tile {
    int ra, rb, bn, kbs, wgs;
    double us[3], extra, call;
};
constexpr Tile TILES[] = {{1, 1, 64, 8, 3, {0.327, 0.382, 0.517}, 5.2, 3.2},
                          {1, 2, 128, 4, 3, {0.250, 0.291, 0.398}, 8.8, 2.8},
                          {2, 1, 64, 4, 3, {0.283, 0.359, 0.448}, 8.6, 2.8},
                          {2, 2, 128, 4, 2, {0.374, 0.486, 0.486}, 9.0, 2.5},
                          {2, 1, 32, 4, 3, {0.248, 0.269, 0.333}, 8.5, 2.9}};
// fp32: the matrix instructions are the limit (70 layers, 20 %)
constexpr Tile TILES32[] = {{1, 1, 64, 8, 3, {0.757, 1.133, 1.622}, 2.4, 2.3},
                            {1, 2, 128, 4, 3, {0.705, 1.116, 1.553}, 3.2, 2.8},
                            {2, 1, 64, 4, 3, {0.687, 1.198, 1.548}, 3.5, 3.0},
                            {2, 2, 128, 4, 2, {1.174, 2.081, 2.081}, 3.0, 3.6},
                            {2, 1, 32, 4, 3, {0.470, 0.713, 0.932}, 3.8, 2.8}};

}  // namespace

MidEstimate igemm_mid_best(const ConvShape* f, int n, size_t room)
{
    const ConvShape& s = f[0];
    const int kpt = padded_k_blocks(s), cols = s.M * s.D3;
    const double out_bytes = 4.0 * (s.out_view ? (double)s.out_alloc : (double)s.out_elems());
    MidEstimate best{{0, 1}, 1e30};
    for (int t = 0; t < 5; ++t) {
        const Tile& tl = s.dtype == 0 ? TILES32[t] : TILES[t];
        if ((tl.bn == 32 && cols > 96) || (tl.bn == 128 && cols <= 64)) continue;
        // (a launch-bound call waits for this: rows and stages of the phases once per tile, and no more
        // pieces once they have made it slower)
        int row_tiles[MAX_PHASES], stages_of[MAX_PHASES];
        double tiles = 0, work = 0, tile_best = 1e30;
        for (int i = 0; i < n; ++i) {
            row_tiles[i] = (int)((unsigned)(f[i].pixels() * s.D1 + 64 * tl.ra - 1) / (64u * tl.ra));
            stages_of[i] = (int)((unsigned)(f[i].kh * f[i].kw * kpt + tl.kbs - 1) / (unsigned)tl.kbs);
            tiles += row_tiles[i];
            work += (double)row_tiles[i] * stages_of[i];
        }
        const double across = (double)((cols + tl.bn - 1) / tl.bn) * s.D0, per_split = tiles * across;
        const double round = 256.0 * tl.wgs, rate = 0.95 * tl.us[tl.wgs - 1] / round;
        for (int nsplit = 1; nsplit <= 32; nsplit += nsplit < 4 ? 1 : nsplit / 2) {
            // (this and more pieces take so long at least: a workgroup's set-up, or all of them at the full chip's rate)
            const double least = std::max(tl.extra * tl.us[0], (work * across + per_split * nsplit * tl.extra) * rate) +
                                 tl.call + (nsplit > 1 ? 3.0 + nsplit * out_bytes * 2.5e-7 : 0.0);
            if (least >= best.us || (nsplit > 1 && nsplit * out_bytes > (double)room)) break;
            int most = 0;
            double sum = 0;
            for (int i = 0; i < n; ++i) {
                const int st = (stages_of[i] + nsplit - 1) / nsplit;
                sum += (double)row_tiles[i] * st;
                if (st > most) most = st;
            }
            if (nsplit > 1 && most < 2) break;
            const double stages = sum / tiles, blocks = per_split * nsplit;
            const double full = (double)(long long)(blocks / round), rest = blocks - full * round;
            double us = tl.call + full * (stages + tl.extra) * tl.us[tl.wgs - 1];
            if (rest > 0)
                us += ((full > 0 ? stages : (double)most) + tl.extra) * tl.us[(int)((rest + 255) / 256) - 1];
            if (nsplit > 1) us += 3.0 + nsplit * out_bytes * 2.5e-7;
            if (us < best.us) best = {{t, nsplit}, us};
            if (us < tile_best) tile_best = us;
            if (blocks >= 1024 || (nsplit > 2 && us > 1.1 * tile_best)) break;
        }
    }
    if (s.mid_use == 2) best.pick = asked_pick(s, best.pick, 5, out_bytes, room);
    return best;
}

namespace {

MidPlan mid_plan(const ConvShape* f, int n, size_t kernel_elems, MidPick pick)
{
    MidPlan pl{};
    MidParams<MAX_PHASES>& P = pl.P;
    const ConvShape& s = f[0];
    const Strides k = kernel_strides(s);
    const int es = elem_size(s), row = s.D2 * es / 2;  // capsule rows in units of 2 bytes
    pl.wide = row % 8 == 0;
    pl.kt = !s.in_gradient;
    P.in_bytes = (unsigned)(s.in_elems() * es);
    P.k_bytes = (unsigned)(kernel_elems * es);
    P.H = s.H; P.W = s.W; P.stride = s.stride; P.D1 = s.D1; P.C = s.C; P.D0 = s.D0;
    P.in_sd0 = s.D1 * s.D2 * es;
    P.pix_bytes = s.C * s.D0 * P.in_sd0;
    P.d1_bytes = s.D2 * es;
    P.in_blk = 16;
    P.kb_shift = pl.wide ? log2_of(row / 8) : 0;
    P.kb_mask = (1 << P.kb_shift) - 1;
    P.in_kb = s.D0 * P.in_sd0 * (pl.wide ? 1 : 2);
    P.kq = k_blocks(s);
    pl.g = mid_group(s);
    P.kpt = padded_k_blocks(s);
    P.kpt_magic = P.kpt == 1 ? 0u : (unsigned)(((1ull << 32) + P.kpt - 1) / P.kpt);
    P.k_sp = (int)(k.sp * es); P.k_sq = (int)(k.sq * es); P.k_sd0 = (int)(k.sd0 * es);
    P.k_sm = (int)(k.sm * es); P.k_c2 = (int)(k.sc * es);
    P.k_kb = (int)(k.sc * es) * (pl.wide ? 1 : 2);
    P.k_blk = (int)(k.sd2 * 16);  // the values of a 16-byte K block times es
    P.k_col = (int)((pl.kt ? k.sd2 : k.sd3) * es);
    P.dc_shift = log2_of(s.D3);
    P.cols = s.M * s.D3;
    P.nphase = n;
    P.by_d1 = fast_div(s.D1);
    P.out_sm = s.D0 * s.D1 * s.D3;
    P.out_sd0 = s.D1 * s.D3;
    const long long pix = (long long)s.M * P.out_sm;
    P.out_sy = s.out_view ? s.out_sy : pix;
    P.out_sx = s.out_view ? s.out_sx : pix * s.Wo;
    P.out_sn = s.out_view ? s.out_sn : pix * s.Wo * s.Ho;
    P.out_elems = s.out_view ? s.out_alloc : (long long)s.out_elems();
    const Tile& tl = TILES[pick.tile];  // (the same shapes for both)
    pl.ra = tl.ra;
    pl.rb = tl.rb;
    pl.wc = tl.bn == 32 ? 1 : 2;
    P.col_tiles = ceil_div(P.cols, tl.bn);
    const int kbs = tl.kbs;
    int row_tiles = 0;
    for (int i = 0; i < n; ++i) {
        const ConvShape& g = f[i];
        MidPhase& F = P.ph[i];
        F.Ho = g.Ho; F.Wo = g.Wo; F.kw = g.kw; F.pad_h = g.pad; F.pad_w = g.padw();
        F.kbs = g.kh * g.kw * P.kpt;
        F.rows = (int)(g.pixels() * s.D1);
        F.tile0 = row_tiles;
        row_tiles += ceil_div(F.rows, 64 * pl.ra);
        F.kw_magic = g.kw <= 1 ? 0 : (int)(unsigned)(((1ull << 32) + g.kw - 1) / g.kw);
        F.by_wo = fast_div(g.Wo);
        F.by_ho = fast_div(g.Ho);
        F.k_base = (int)(g.kernel_view ? g.k_base * es : 0);
        F.out_base = g.out_view ? g.out_base : 0;
    }
    const long long tiles = (long long)row_tiles * P.col_tiles * s.D0;
    P.tiles = (int)tiles;
    const int nsplit = pick.nsplit;
    P.nsplit = nsplit;
    for (int i = 0; i < n; ++i) P.ph[i].stages_per_split = ceil_div(ceil_div(P.ph[i].kbs, kbs), nsplit);
    pl.blocks = tiles * nsplit;
    P.xcd_per = (int)(pl.blocks / 8);
    pl.out16 = s.out16 != 0 && nsplit == 1;  // (with a split the reduction rounds)
    return pl;
}

template <typename Tag, bool WIDE, int G, bool KT, bool OUT16, int RA, int RB, int WC, int KBS, int NST>
hipError_t launch_tile(const MidPlan& pl, hipStream_t stream)
{
    constexpr int lds = NST * KBS * (RA + RB) * 1024;
    auto kern = igemm_mid_kernel<Tag, WIDE, G, KT, OUT16, RA, RB, WC, KBS, NST>;
    static std::atomic<unsigned long long> lds_set{0};
    const hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), lds, lds_set);
    if (err != hipSuccess) return err;
    if constexpr (KT)
        kern<<<dim3((unsigned)pl.blocks), dim3(256), lds, stream>>>({pl.P, {pl.P.ph[0]}});
    else
        kern<<<dim3((unsigned)pl.blocks), dim3(256), lds, stream>>>(pl.P);
    return hipGetLastError();
}
template <typename Tag, bool WIDE, int G, bool KT, bool OUT16>
hipError_t launch_mode(const MidPlan& pl, hipStream_t stream)
{
    // 64x64: 16 KB stages of 64 K values, three of them: three workgroups per CU (eight
    // stages and one workgroup: no faster).  Larger tiles: stages of 32 K values (12 or 16 KB), four of
    // them: three or two workgroups
    if (pl.wc == 1) return launch_tile<Tag, WIDE, G, KT, OUT16, 2, 1, 1, 4, 4>(pl, stream);
    if (pl.ra == 2)
        return pl.rb == 2 ? launch_tile<Tag, WIDE, G, KT, OUT16, 2, 2, 2, 4, 4>(pl, stream)
                          : launch_tile<Tag, WIDE, G, KT, OUT16, 2, 1, 2, 4, 4>(pl, stream);
    if (pl.rb == 2) return launch_tile<Tag, WIDE, G, KT, OUT16, 1, 2, 2, 4, 4>(pl, stream);
    return launch_tile<Tag, WIDE, G, KT, OUT16, 1, 1, 2, 8, 3>(pl, stream);
}
template <typename Tag, bool WIDE, int G>
hipError_t launch_out(const MidPlan& pl, hipStream_t stream)
{
    if (pl.kt) return pl.out16 ? launch_mode<Tag, WIDE, G, true, true>(pl, stream)
                               : launch_mode<Tag, WIDE, G, true, false>(pl, stream);
    return pl.out16 ? launch_mode<Tag, WIDE, G, false, true>(pl, stream)
                    : launch_mode<Tag, WIDE, G, false, false>(pl, stream);
}
template <typename Tag>
hipError_t launch_tag(const MidPlan& pl, hipStream_t stream)
{
    if (!pl.wide) return launch_out<Tag, false, 2>(pl, stream);
    return pl.g == 4   ? launch_out<Tag, true, 4>(pl, stream)
           : pl.g == 2 ? launch_out<Tag, true, 2>(pl, stream)
                       : launch_out<Tag, true, 1>(pl, stream);
}

template <int G>
hipError_t launch_f32_group(const MidPlan& pl, hipStream_t stream)
{
    return launch_mode<f32_tag, true, G, false, false>(pl, stream);
}
hipError_t launch_f32(const MidPlan& pl, hipStream_t stream)
{
    return pl.g == 4   ? launch_f32_group<4>(pl, stream)
           : pl.g == 2 ? launch_f32_group<2>(pl, stream)
                       : launch_f32_group<1>(pl, stream);
}

}  // namespace

// Shapes the kernel can run.  `f`: n phases of one input gradient, or one forward pass or input
// gradient (kernel tensor dense in the forward pass, a view with contiguous K values otherwise).
bool igemm_mid_eligible(const ConvShape* f, int n, size_t kernel_elems)
{
    const ConvShape& s = f[0];
    if (n < 1 || n > MAX_PHASES || s.in_paired || s.mid_use == 1) return false;
    if (s.in_gradient && (!s.kernel_view || s.k_sd2 != 1)) return false;  // (reads 16 bytes of K values)
    if (s.H > MAX_EXTENT || s.W > MAX_EXTENT || s.stride > MAX_EXTENT) return false;
    if (!pow2(s.D3) || s.D3 < 4) return false;  // 4 consecutive columns per lane, shifts
    if (s.dtype == 0) {
        if (!s.in_gradient || !pow2(s.D2) || s.D2 < 4) return false;
    } else if (s.D2 % 8 == 0) {
        if (!pow2(s.D2) || (!s.in_gradient && s.D3 % 8 != 0)) return false;
    } else if (s.D2 != 4 || s.D1 % 2 != 0 || (!s.in_gradient && s.D3 != 4)) {
        return false;
    }
    const size_t es = elem_size(s);
    if (s.in_elems() * es >= MAX_TENSOR_BYTES || kernel_elems * es >= MAX_TENSOR_BYTES) return false;
    const bool cols_ok = (long long)s.M * s.D3 < (1LL << 24);
    const long long kpt = (long long)s.C * (s.D2 * es < 16 ? 1 : s.D2 * es / 16) + 3;
    for (int i = 0; i < n; ++i) {
        const long long rows = f[i].pixels() * s.D1, kbs = (long long)f[i].kh * f[i].kw * kpt;
        if (rows >= (1LL << 30) || f[i].out_sn < 0 || f[i].out_sx < 0 || f[i].out_sy < 0) return false;
        // divisions by multiplication: exact while dividend times divisor stays below 2^32
        if ((kbs + 1024) * kpt >= (1LL << 32) || (kbs + 1024) * f[i].kw >= (1LL << 32)) return false;
        // and no tap position of the K loop's end may meet an image row
        if (f[i].kw > MAX_EXTENT || f[i].kh > MAX_EXTENT || f[i].pad >= MAX_EXTENT / 2 ||
            f[i].padw() >= MAX_EXTENT / 2 || s.H > MAX_EXTENT / 2)
            return false;
    }
    return cols_ok;
}

// Estimated time of the 16-bit kernels with 256-row tiles on a convolution, us: fits over the layers of a random
// sample (0.003 .. 600 GFLOP, forward and input gradient) that these kernels served, 45 and 168 of them,
// within 21 % root mean square.  A call, the FLOPs of whole tiles at a rate of the capsule shape's, and
// the bytes of input and output, the input three times where its channels are paired first.
double igemm16_tuned_us(const ConvShape& s, MfmaKernel which)
{
    const bool fast = which == MfmaKernel::Tuned16, four = s.D2 == 4;
    const long long cols = (long long)s.M * s.D3;
    const long long bn = fast ? 256 : cols < 128 ? (cols + 31) / 32 * 32 : 128;
    const double gflop = 2e-9 * (double)((s.pixels() * s.D1 + 255) / 256 * 256) *
                         (double)((cols + bn - 1) / bn * bn) * s.D0 * s.kh * s.kw * s.C * s.D2;
    const double in_mb = 2e-6 * (double)s.in_elems(), out_mb = (s.out16 ? 2e-6 : 4e-6) * (double)s.out_elems();
    if (fast) return 12.8 + gflop / 1.48 + 0.14 * (in_mb + out_mb);
    if (four) return 17.4 + gflop / 1.22 + 0.17 * (3 * in_mb + out_mb);
    if (s.D1 <= 2) return 19.5 + gflop / 0.72 + 0.12 * (in_mb + out_mb);
    return 11.2 + gflop / 1.01 + 0.13 * (in_mb + out_mb);
}

// Measured with and without this kernel over random layers, 1500 of them 16-bit forward passes and input gradients.
// Against the any-shape kernel (three launches) always: 800 layers, none slower, 0.5 times its
// time on average.  Against the small-problem kernel (360 layers, 0.56 times) but for one tile or two of a long K
// loop and next to no work, where that kernel's many short pieces win (2 images, a 5x5 window over 77 channels of
// 4x4: 11.0 against 9.3 us; the fully-connected layer over 8x8 images of 64 channels of 8x8, 0.04 GFLOP, too when called again
// and again, 12.4 against 10.8, but behind four other layers, its kernel tensor in no L2, this one: the stack on two images
// 96.9 against 98.9, on four 139 against 143), and rows of 4 of one channel or two under few columns, whose K blocks (pairs of two
// channels) and 64-column tiles are mostly padding: 300 layers of 4x4 of 0.05 MFLOP and more, called again and again / with
// cold caches, 85 stay there, which take 1.14 / 1.06 times the time here (one channel, a 5x5 window, 12 columns: 5.6 against
// 3.7 / 4.2 us; 3x3, 8 columns: 4.0 against 3.1 / 3.3); of the others none loses more than 3 % with cold caches.  Against the kernels of
// 256-row tiles where the estimates differ by 35 % (508 layers, 81 leave, for 0.2 .. 0.9 of the time; by 30 % and without the next sentence
// 124, three of them 4 .. 22 % slower; by 20 % 179, five).  An input that no cache holds takes its time
// whatever the tiles, 0.3 us per MB: 198 images of 13x39 with 49 channels at stride 2, 0.63 GB, 184 us, not the
// estimate's 82; 99 of 36x36 with 16 channels of 16x16, 1.05 GB, 414.
// fp32 input gradients: against the small-problem and the any-shape kernel, which read the kernel tensor
// through strides or after a repack pass, from 24 columns on, but for a few tiles of a long K loop (28 random layers 0.41 .. 0.85 times the time, one
// of 5.6 us 0.3 us slower; at 24 columns five 0.63 .. 1.06; 8 and 16 columns 1.13 and 1.2 times); against the kernel on bf16 instructions where
// the estimates differ by a quarter.
MidPick igemm_mid_choice(const ConvShape& s, MfmaKernel otherwise, size_t room)
{
    if ((s.dtype == 0 && !s.in_gradient) || !igemm_mid_eligible(&s, 1, s.kernel_elems())) return {};
    if (s.mid_use == 2) return igemm_mid_best(&s, 1, room).pick;
    const double flops = 2.0 * (double)s.out_elems() * s.kh * s.kw * s.C * s.D2;
    const bool tuned = otherwise != MfmaKernel::Generic && otherwise != MfmaKernel::Small;
    if (s.dtype == 0 && (tuned ? otherwise != MfmaKernel::Dma32 : (long long)s.M * s.D3 < 24)) return {};
    if (otherwise == MfmaKernel::Small && !s.in_gradient && s.D2 == 4 && s.C <= 2 && s.C * s.M * s.D3 <= 48 &&
        s.kh * s.kw * s.C * s.D2 <= 200)
        return {};
    const MidEstimate e = igemm_mid_best(&s, 1, room);
    bool take;
    if (s.dtype == 0)
        take = tuned ? e.us < 0.75 * igemm32_us(s, otherwise) : flops >= 1e8 || e.us < 12;
    else if (tuned)
        take = std::max(e.us, 6e-7 * (double)s.in_elems()) < 0.65 * igemm16_tuned_us(s, otherwise);
    else
        take = otherwise == MfmaKernel::Generic || e.us <= 9.5 || flops >= 3e7;
    return take ? e.pick : MidPick{};
}

hipError_t launch_igemm_mid(const ConvShape* f, int n, size_t kernel_elems, MidPick pick, const void* in,
                            const void* kernel, float* out, void* workspace, hipStream_t stream, bool skip_taps)
{
    if (skip_taps) pick.nsplit = 1;  // (partial sums cannot tell)
    MidPlan pl = mid_plan(f, n, kernel_elems, pick);
    pl.P.skip_taps = skip_taps;
    pl.P.in = in;
    pl.P.kernel = kernel;
    float* partial = static_cast<float*>(workspace);
    pl.P.out = pl.P.nsplit > 1 ? partial : out;
    const hipError_t err = f[0].dtype == 0   ? launch_f32(pl, stream)
                           : f[0].dtype == 1 ? launch_tag<bf16_tag>(pl, stream)
                                             : launch_tag<f16_tag>(pl, stream);
    if (err != hipSuccess || pl.P.nsplit == 1) return err;
    return launch_splitk_reduce(partial, out, pl.P.out_elems, pl.P.nsplit, stream, f[0].out16);
}

}  // namespace capscaps
