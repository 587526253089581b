// fp32 matrix-core kernel of the capsule convolution forward pass on the 16-bit matrix units.
// Same implicit GEMM as the other igemm kernels (rows (pixel,d1), columns (m,d3),
// K = (tap, c, d2); paper Algorithm 2), for capsule rows of 3k or 4k floats.
//
// Bound: the matrix rate.  The fp32 matrix instructions of this chip run at a sixteenth of the
// bf16 ones (157 against 2517 TFLOP/s), so every fp32 value is written, times 2^23, as the exact sum
// of three bf16 values (bf16_split.h).  A product is then nine bf16 products, each exact in the fp32 accumulator; the six with
// i + j <= 4 are added up, smallest first, and the three left out (x2 y3, x3 y2, x3 y3) are below
// 2^-25 of the product, less than the rounding of one fp32 addition.  Six instructions for 16 K
// values take 192 cycles per 32 x 32 tile where the fp32 ones take 512.  The sums themselves
// stay in fp32, with fewer roundings (6 accumulations per 16 K values, not 8).  The bf16 instructions
// drop what lies far below the accumulator's last bit toward minus infinity, which in a long K loop
// adds up; the accumulators and the input values change sign every FLIP stages, so that the dropped
// parts cancel.  Root mean square error against 64-bit sums (results of size 1) at K = 1152, 9600,
// 55296, 131072: fp32 instructions 6.1e-7, 1.8e-6, 4.2e-6, 6.5e-6, here 5.2e-7, 1.5e-6, 3.2e-6,
// 4.7e-6, mean errors below 6e-8 (without the sign change 5.2e-7, 1.6e-6, 4.1e-6, 6.9e-6, of that
// -6e-8, -4.9e-7, -2.3e-6, -4.8e-6 in one direction).
//
// Measured (N = 64, 32x32, 3x3, 32 -> 32 channels): 3x3x3 capsules 0.776 ms on the fp32
// instructions, 0.522 ms here (error against 64-bit sums 5.2e-7 and 4.4e-7), 4x4 capsules 0.664
// and 0.333 ms, 8x8 capsules 4.37 and 2.55 ms (232 TFLOP/s).  With the splitting on the matrix cores' pipe (minus_bf16
// in the place of minus_low) 0.543, 0.348 and 2.68 ms.  The long K loops run at the clock the
// power limit leaves (1.5 .. 1.6 GHz); 3-float chunks also at the rate of the L1 lookups (57 per
// copy, 16 where 4-float rows lie side by side).
//
// What the decomposition cannot represent is recomputed: infinities, NaNs, values of 2^104 and more
// and sums of 2^82 and more make their sums infinite or NaN.  A workgroup that finds a sum that is
// not finite runs its K loop again on the fp32 matrix instructions from the same LDS data (the
// input side lies there unsplit; the kernel side's three terms give the fp32 value exactly).
//
// Unit of data movement on the input side: a 16-byte LDS slot holding CW = 3 or 4 consecutive d2
// of one capsule row ("chunk"); a 3-float chunk is copied by a 12-byte buffer load, which lands at
// a 16-byte lane stride.  A stage of the K loop is 4 slots of every row.  The lower half wave
// takes slots 0 and 1 of its row, the upper half slots 2 and 3: 8 values (CW = 4), the K extent of
// one bf16 instruction, or 6 (CW = 3), so that four stages make three instructions' worth.  The
// values are split in registers (6.5 vector instructions each, under the matrix instructions of the
// SIMD's other wave); the kernel tensor is split once per call, by the repack pass.
//
// Tile: 64*NW rows x 32*TN columns; wave w copies and contracts rows 64w..64w+63 (two MFMA row
// tiles) against all TN column tiles, so no input value is split twice in a workgroup.  Lane i of
// a wave copies row 64w+i: its byte offset, with the out-of-range mark where the current tap
// falls into the padding, sits in one VGPR and is refreshed once per stage from a per-lane bit
// mask over the taps; everything else (tap, channel group, chunk) is a scalar offset.  K runs
// channel group outermost, tap inside; ring of NB LDS stages, one barrier per stage; the K loop
// can be split over blocks (partial sums are reduced in a fixed order by the caller's kernel).
#include <hip/hip_runtime.h>

#include "bf16_split.h"
#include "igemm_common.h"
#include "lds_dma.h"

namespace capscaps {
namespace {

constexpr int SLOTS = 4;  // input-side slots per row and stage
// Stages the K loop's body covers: with 3-float chunks four, after which the K values of both half
// waves are whole instructions again, with 4-float ones two, so that the split values of a stage
// and of the next one have registers of their own.
constexpr int stage_period(int cw) { return cw == 3 ? 4 : 2; }
// Ring depths.  A stage's input values are read from LDS and split one stage ahead of their use.
// Two four-wave workgroups share a CU (80 KB each): three input stages of 16 KB and three kernel
// stages of 3 KB per column tile, or two where four column tiles leave room for no more (the
// first operands of a stage are then read at its beginning, not at the end of the one before).
constexpr int NBA = 3;
constexpr int kernel_ring(int tn) { return tn == 4 ? 2 : 3; }

// Columns of a tile.  TRIPLE (D3 a multiple of 3): a lane's accumulator registers of one output row, 16
// per column tile, hold whole runs of three consecutive columns, so that a capsule row is stored
// 12 bytes at a time: half wave h holds the 3 * runs columns from h * 3 * runs on (with three column
// tiles all 48 registers, else one or two less).  Otherwise columns and registers are in the
// order of the matrix instruction: 8g + 4h + i in registers 4g + i.
constexpr int column_runs(int tn) { return 16 * tn / 3; }
constexpr int tile_columns(bool triple, int tn) { return triple ? 6 * column_runs(tn) : 32 * tn; }

template <int CW, int TN, int NW, bool TRIPLE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 4 ? 2 : 1)))
void igemm32_split_kernel(const Dma32Params P)
{
    constexpr int PER = stage_period(CW), NBB = kernel_ring(TN);
    constexpr bool AHEAD = NBB == 3;  // the first kernel operands are read one stage ahead
    constexpr int BM = 64 * NW, BN = 32 * TN, TM = 2;
    constexpr int A_BYTES = SLOTS * BM * 16, B_BYTES = 3 * 2 * BN * 16;
    constexpr int B_LDS = NBA * A_BYTES;              // kernel-side ring after the input-side one
    constexpr int SHARE = B_BYTES / NW;               // kernel-side bytes a wave copies per K step
    constexpr int BPW = (SHARE + 1023) / 1024;        // ... in copies of at most 64 lanes
    constexpr int LAST_LANES = SHARE / 16 - 64 * (BPW - 1);
    constexpr int NPAIR = TM * CW;                    // pairs of input values to split per stage
    constexpr int WORDS = PER * CW;                   // pairs per row tile and period
    constexpr int OOB = (int)0x80000000u;

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
    const int col0 = col_tile * tile_columns(TRIPLE, TN);

    // ---- this lane's row: byte offset of its capsule row in the window's first input pixel,
    // relative to the first image the tile touches, and the bit mask of taps that read a real
    // input pixel
    const int hw = P.Ho * P.Wo;
    // (64-bit divisions only where the row count needs them: they are long)
    const long long n_first = P.rows < (1LL << 31) ? (long long)((unsigned)row0 / (unsigned)(hw * P.D1))
                                                   : row0 / ((long long)hw * P.D1);
    const int row_rel0 = (int)(row0 - n_first * hw * P.D1);  // the tile's first row within that image
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
        const int r = 64 * wave + lane;
        const bool exists = row0 + r < P.rows;
        const unsigned rr = (unsigned)(row_rel0 + (exists ? r : 0));
        const unsigned pixel = rr / (unsigned)P.D1;  // from image n_first on
        const int d1 = (int)(rr - pixel * P.D1);
        const int n_rel = (int)(pixel / (unsigned)hw);
        const int rem = (int)pixel - n_rel * hw;
        const int x = (int)((unsigned)rem / (unsigned)P.Wo), y = rem - x * P.Wo;
        const int ih0 = x * P.stride - P.pad, iw0 = y * P.stride - P.pad_w;
        row_off = (int)((((long long)n_rel * P.H + ih0) * P.W + iw0) * pix_bytes) +
                  (d0 * P.D1 + d1) * P.D2 * 4 + bias;
        // taps q with 0 <= iw0 + q < W, then the window rows inside the image
        const int q_lo = iw0 < 0 ? -iw0 : 0, q_hi = P.W - iw0 < P.kw ? P.W - iw0 : P.kw;
        unsigned long long row_taps = 0;
        if (exists && q_hi > q_lo)
            row_taps = (q_hi >= 64 ? ~0ull : (1ull << q_hi) - 1) & ~((1ull << q_lo) - 1);
        for (int p = 0; p < P.kh; ++p)
            if ((unsigned)(ih0 + p) < (unsigned)P.H) tap_ok |= row_taps << (p * P.kw);
    }
    long long in_left = P.in_bytes - n_first * img_bytes + bias;
    if (in_left > 0x7fffffffLL) in_left = 0x7fffffffLL;
    const rsrc_t rs_in = make_rsrc(in_base, (unsigned)in_left);
    const rsrc_t rs_kp = make_rsrc(P.kp, (unsigned)P.kp_bytes);
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;

    // ---- K loop state of the next stage to copy (all scalar)
    const int st_begin = split * P.stages_per_split;  // a multiple of PER
    int st_end = st_begin + P.stages_per_split;
    if (st_end > P.nstages) st_end = P.nstages;
    const int my_stages = st_end - st_begin;
    const int chan_per_group = SLOTS / P.D2C;                // D2C is 1, 2 or 4
    const int g_step = chan_per_group * P.cs * 4;           // bytes per channel group
    const int row_skip = (P.W - P.kw + 1) * pix_bytes;
    int issued, tap, tap_q, tap_off, g_off, c0, kp_off;
    int q_off[SLOTS], q_chan[SLOTS];
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
        q_chan[q] = q / P.D2C;
        q_off[q] = (q_chan[q] * P.cs + (q % P.D2C) * CW) * 4;
    }
    const unsigned b_voff = (unsigned)(wave * SHARE + lane * 16);

    auto restart = [&]() {
        issued = 0;
        tap = st_begin % P.ntaps;
        const int grp = st_begin / P.ntaps;
        tap_q = tap % P.kw;
        tap_off = ((tap / P.kw) * P.W + tap_q) * pix_bytes;
        g_off = grp * g_step;
        c0 = grp * chan_per_group;  // first channel of the group
        kp_off = (int)((((long long)d0 * P.col_tiles + col_tile) * P.ksteps +
                        (CW == 3 ? st_begin / 4 * 3 : st_begin)) * B_BYTES);
    };
    // input copies of the next stage into the ring slot at LDS address `slot`: this lane's row ...
    unsigned a_voff;
    auto begin_a = [&]() {
        // (no branch: it would cut the stage's one basic block; 5x5 window, 20 images of 31x27, 20 -> 14 channels of
        // 6x5 . 5x4, 211.4 -> 209.0 us, its input gradient 196.7 -> 193.9; 3x3x3 layers 524.8 -> 522.1)
        const unsigned live = issued < my_stages ? 1u : 0u;
        a_voff = ((unsigned)(tap_ok >> tap) & live) != 0 ? (unsigned)row_off : (unsigned)OOB;
    };
    // ... its slot q
    auto copy_a = [&](unsigned slot, int q) {
        const bool chan_ok = c0 + q_chan[q] < P.C;  // last group may be partial
        copy_to_lds_dwords<CW>(rs_in, slot + (q * BM + 64 * wave) * 16,
                               chan_ok ? a_voff : (unsigned)OOB, tap_off + g_off + q_off[q]);
    };
    // next stage: next tap, after the last tap the next channel group (selects, no branches)
    auto advance_a = [&]() {
        ++issued;
        ++tap;
        ++tap_q;
        const bool row_end = tap_q == P.kw, wrap = tap == P.ntaps;
        tap_q = row_end ? 0 : tap_q;
        tap_off = wrap ? 0 : tap_off + (row_end ? row_skip : pix_bytes);
        tap = wrap ? 0 : tap;
        g_off += wrap ? g_step : 0;
        c0 += wrap ? chan_per_group : 0;
    };
    // kernel copy j of this wave's share of the next K step
    auto copy_b = [&](unsigned slot, auto J) {
        constexpr int j = decltype(J)::value;
        if constexpr (j < BPW - 1 || LAST_LANES == 64)
            copy_to_lds_dwords<4>(rs_kp, slot + wave * SHARE + j * 1024, b_voff, kp_off + j * 1024);
        else
            copy_to_lds_16B_lanes(rs_kp, slot + wave * SHARE + j * 1024, b_voff, kp_off + j * 1024,
                                  (1ull << (LAST_LANES & 63)) - 1);
    };
    auto has_step = [](int pos) constexpr { return CW == 4 || (pos + 8) % PER != 0; };

    float16v acc[TN][TM];
    auto clear_acc = [&]() {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    };
    const unsigned a_rd = (unsigned)((2 * h * BM + 64 * wave + lr) * 16);
    const unsigned b_rd = (unsigned)((h * BN + lr) * 16);
    auto read_kernel = [&](const char* slot, int a, int t) -> chunk_t {
        return *reinterpret_cast<const chunk_t*>(slot + b_rd + (2 * t * BN + a * 32) * 16);
    };
    auto read_input = [&](const char* slot, int b, int u) -> float4v {
        return *reinterpret_cast<const float4v*>(slot + a_rd + (u * BM + b * 32) * 16);
    };

    // ---- the K loop on the split values
    {
        constexpr int FLIP = 96;  // stages; a multiple of both periods
        // One-wave workgroups are at most one per SIMD (Dma32Plan::nw): with one column tile, splitting as many values for
        // the fewest matrix instructions, their wave's issue is the limit, and dot products take the remainders.  10
        // random layers 0.94 .. 0.98 of the time of subtractions (47 -> 5 channels of 4x8 . 8x4, 19 images of 29x29, 106.6 ->
        // 100.2 us); with two column tiles 0.99 .. 1.03 (11 layers), with three and four 1.01 .. 1.09 (20), four-wave
        // workgroups 0.98 .. 1.10 (119).
        constexpr bool DOT = NW == 1 && TN == 1;
        const MinusOne one;
        // of the input values being split; the ranges of a split K loop begin with either sign
        unsigned in_scale = __builtin_bit_cast(unsigned, SPLIT_SCALE) | (unsigned)split << 31;
        // K values of one period, split: pairs per row tile and term
        unsigned iv[TM][3][WORDS];
        float lo[NPAIR], hi[NPAIR];  // the pairs being split: what the terms so far leave over
        // step `k` (0 .. SPLIT_STEPS - 1) of splitting pair `p` of a stage at place `pos` of the period
        auto split_step = [&](int p, int k, int pos) {
            unsigned(&w)[3][WORDS] = iv[p / CW];
            const int at = pos * CW + p % CW, t = (k - 2) / 3;
            if (k == 0)
                lo[p] *= __builtin_bit_cast(float, in_scale);
            else if (k == 1)
                hi[p] *= __builtin_bit_cast(float, in_scale);
            else if (k % 3 == 2)
                w[t][at] = round_pair(lo[p], hi[p]);
            else if (k % 3 == 0)
                lo[p] = DOT ? minus_bf16(lo[p], w[t][at], one.lo) : minus_low(lo[p], w[t][at]);
            else
                hi[p] = DOT ? minus_bf16(hi[p], w[t][at], one.hi) : minus_high(hi[p], w[t][at]);
        };
        auto take_input = [&](const char* slot) {
            float4v raw[TM][2];
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int u = 0; u < 2; ++u) raw[b][u] = read_input(slot, b, u);
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int i = 0; i < CW; ++i) {
                    lo[b * CW + i] = raw[b][2 * i / CW][2 * i % CW];
                    hi[b * CW + i] = raw[b][(2 * i + 1) / CW][(2 * i + 1) % CW];
                }
        };
        clear_acc();
        restart();
        // prologue: kernel side of the first NBB-1 stages, input side of three, all but the last
        // input stage landed; the first stage's input split
        static_for<NBB - 1>([&](auto S0) {
            constexpr int s0 = decltype(S0)::value;
            if constexpr (has_step(s0)) {
                static_for<BPW>([&](auto J) { copy_b(lds0 + B_LDS + s0 * B_BYTES, J); });
                kp_off += B_BYTES;
            }
        });
        static_for<NBA>([&](auto S0) {
            begin_a();
#pragma unroll
            for (int q = 0; q < SLOTS; ++q) copy_a(lds0 + decltype(S0)::value * A_BYTES, q);
            advance_a();
        });
        __builtin_amdgcn_s_waitcnt(0x0F70 | SLOTS);
        __syncthreads();
        take_input(smem);
#pragma unroll
        for (int k = 0; k < SPLIT_STEPS; ++k)
#pragma unroll
            for (int p = 0; p < NPAIR; ++p) split_step(p, k, 0);
        chunk_t kb[2][3];  // kernel operands of a column tile, double-buffered
        if constexpr (AHEAD && has_step(0)) {
#pragma unroll
            for (int t = 0; t < 3; ++t) kb[0][t] = read_kernel(smem + B_LDS, 0, t);
        }
        // the input slot of stage 0, just read, takes stage 3
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __syncthreads();
        // ring slots (byte offsets): input of the next stage (read) and of the one three ahead
        // (copied into: this stage's own slot), kernel of this stage and of the next
        unsigned a_next = A_BYTES, a_cur = 0, b_cur = B_LDS;
        int to_flip = FLIP;
        for (int st = 0; st < my_stages; st += PER) {
            if (to_flip == 0) {
                to_flip = FLIP;
                in_scale ^= 0x80000000u;
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b) acc[a][b] = -acc[a][b];
                // the input values of the stage at hand, a period's first, are split already
#pragma unroll
                for (int b = 0; b < TM; ++b)
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int i = 0; i < CW; ++i) iv[b][t][i] ^= 0x80008000u;
            }
            to_flip -= PER;
            static_for<PER>([&](auto POS) {
                constexpr int pos = decltype(POS)::value, next = (pos + 1) % PER;
                constexpr int NMMA = has_step(pos) ? TN * TM * 6 : 0;
                constexpr int g = CW == 4 ? pos : pos - 1;  // K step within the period
                constexpr int W0 = 4 * g;                    // its first pair
                const unsigned b_next = b_cur + B_BYTES == B_LDS + NBB * B_BYTES ? B_LDS : b_cur + B_BYTES;
                const unsigned b_after = b_next + B_BYTES == B_LDS + NBB * B_BYTES ? B_LDS : b_next + B_BYTES;
                const unsigned b_fill = NBB == 3 ? b_after : b_next;
                constexpr bool fill = has_step(pos + NBB - 1);
                if constexpr (!AHEAD && NMMA > 0) {
#pragma unroll
                    for (int t = 0; t < 3; ++t) kb[0][t] = read_kernel(smem + b_cur, 0, t);
                }
                take_input(smem + a_next);
                // side operations, dealt out over the gaps after the matrix instructions: the
                // copies, the operands of the next column tile, the next stage's splitting
                constexpr int NSTEP = SPLIT_STEPS * NPAIR, GAPS = NMMA > 0 ? NMMA : 1;
                constexpr int FIRST = NMMA > 0 ? 6 : 0;  // the input values need time to arrive
                static_for<GAPS>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if constexpr (NMMA > 0) {
                        constexpr int a = i / (6 * TM), u = i / TM % 6, b = i % TM;
                        const unsigned(&w)[WORDS] = iv[b][SPLIT_TERM_B[u]];
                        const chunk_t x = {w[W0], w[W0 + 1], w[W0 + 2], w[W0 + 3]};
                        Mma<bf16_tag>::run(kb[a & 1][SPLIT_TERM_A[u]], x, acc[a][b]);
                        // operands of the next column tile, or of the next stage's first
                        constexpr int f = i % (6 * TM) - 1;
                        if constexpr (f >= 0 && f < 3) {
                            if constexpr (a + 1 < TN)
                                kb[(a + 1) & 1][f] = read_kernel(smem + b_cur, a + 1, f);
                        }
                    }
                    constexpr int NSIDE = SLOTS + BPW;
                    constexpr int j0 = dealt_before(i, NSIDE, GAPS, 0), j1 = dealt_before(i + 1, NSIDE, GAPS, 0);
                    static_for<j1 - j0>([&](auto J) {
                        constexpr int j = j0 + decltype(J)::value;
                        if constexpr (j < BPW) {
                            if constexpr (fill) {
                                copy_b(lds0 + b_fill, std::integral_constant<int, j < BPW ? j : 0>{});
                                if constexpr (j == BPW - 1) kp_off += B_BYTES;
                            }
                            if constexpr (j == BPW - 1) begin_a();
                        } else {
                            copy_a(lds0 + a_cur, j - BPW);
                            if constexpr (j == SLOTS + BPW - 1) advance_a();
                        }
                    });
                    constexpr int t0 = dealt_before(i, NSTEP, GAPS, FIRST), t1 = dealt_before(i + 1, NSTEP, GAPS, FIRST);
#pragma unroll
                    for (int t = t0; t < t1; ++t) split_step(t % NPAIR, t / NPAIR, next);
                    if constexpr (NMMA > 0) __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (AHEAD && has_step(next)) {
#pragma unroll
                    for (int t = 0; t < 3; ++t) kb[0][t] = read_kernel(smem + b_next, 0, t);
                }
                // all of this wave's copies but those of the input stage three ahead have landed,
                // its reads are done; after the barrier both hold for every wave
                __builtin_amdgcn_s_waitcnt((0x0F70 | SLOTS) & 0xF0FF);
                __syncthreads();
                a_cur = a_next;
                a_next = a_next + A_BYTES == NBA * A_BYTES ? 0 : a_next + A_BYTES;
                b_cur = b_next;
            });
        }
        // the copies of the surplus stages still write into this workgroup's LDS
        __builtin_amdgcn_s_waitcnt(0x0F70);
        const float unscale = in_scale >> 31 ? -SPLIT_UNSCALE : SPLIT_UNSCALE;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) acc[a][b] *= unscale;
    }

    // ---- the same sums on the fp32 matrix instructions, one stage at a time
    auto contract_exact = [&]() {
        clear_acc();
        restart();
        float ix[TM][2 * WORDS];
        for (int st = 0; st < my_stages; st += PER) {
            static_for<PER>([&](auto POS) {
                constexpr int pos = decltype(POS)::value;
                begin_a();
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) copy_a(lds0, q);
                advance_a();
                if constexpr (has_step(pos)) {
                    static_for<BPW>([&](auto J) { copy_b(lds0 + B_LDS, J); });
                    kp_off += B_BYTES;
                }
                __builtin_amdgcn_s_waitcnt(0x0F70);
                __syncthreads();
#pragma unroll
                for (int b = 0; b < TM; ++b)
#pragma unroll
                    for (int v = 0; v < 2 * CW; ++v)
                        ix[b][2 * CW * pos + v] = read_input(smem, b, v / CW)[v % CW];
                if constexpr (has_step(pos)) {
                    constexpr int V0 = 8 * (CW == 4 ? pos : pos - 1);
#pragma unroll
                    for (int a = 0; a < TN; ++a) {
                        chunk_t k[3];
#pragma unroll
                        for (int t = 0; t < 3; ++t) k[t] = read_kernel(smem + B_LDS, a, t);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            unsigned v[3];
#pragma unroll
                            for (int t = 0; t < 3; ++t)
                                v[t] = e & 1 ? k[t][e / 2] >> 16 : k[t][e / 2] & 0xffffu;
                            const float kv = joined_kernel_value(v[0], v[1], v[2]);
#pragma unroll
                            for (int b = 0; b < TM; ++b)
                                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(kv, ix[b][V0 + e], acc[a][b], 0, 0, 0);
                        }
                    }
                }
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __syncthreads();
            });
        }
    };

    {
        SplitCheck check;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) check.take(acc[a][b]);
        const bool redo = check.failed();
        __syncthreads();  // every wave's copies have landed: LDS is free
        if (lane == 0) reinterpret_cast<int*>(smem)[wave] = 0;
        const unsigned long long any = __builtin_amdgcn_ballot_w64(redo);
        if (lane == 0) reinterpret_cast<int*>(smem)[wave] = any != 0;
        __syncthreads();
        int again = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) again |= reinterpret_cast<const int*>(smem)[w];
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(again)) contract_exact();
    }

    // ---- epilogue
    float* __restrict__ out = P.out + (long long)split * P.out_elems;
    const int caps_out = P.D0 * P.D1 * P.D3;
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const int r = 64 * wave + b * 32 + lr;
        if (row0 + r >= P.rows) continue;
        const unsigned rr = (unsigned)(row_rel0 + r);
        const unsigned pixel = rr / (unsigned)P.D1;  // from image n_first on
        const int d1 = (int)(rr - pixel * P.D1);
        long long pix_at;
        if (P.out_mode & 1) {
            const int n_rel = (int)(pixel / (unsigned)hw);
            const int rem = (int)pixel - n_rel * hw;
            const int x = (int)((unsigned)rem / (unsigned)P.Wo), y = rem - x * P.Wo;
            pix_at = P.out_base + (n_first + n_rel) * P.out_sn + x * P.out_sx + y * P.out_sy;
        } else {
            pix_at = (n_first * hw + pixel) * P.M * caps_out;
        }
        float* orow = out + pix_at + (d0 * P.D1 + d1) * P.D3;
        if constexpr (TRIPLE) {
            // run k of half wave h: columns col0 + 3 (h * RUNS + k) .. + 2, one capsule row piece
            constexpr int RUNS = column_runs(TN);
            struct __attribute__((packed, aligned(4))) run_t { float v[3]; };
            auto run_of = [&](int k) -> run_t {
                run_t t;
#pragma unroll
                for (int i = 0; i < 3; ++i) t.v[i] = acc[(3 * k + i) / 16][b][(3 * k + i) % 16];
                return t;
            };
            const int j0 = col0 + 3 * h * RUNS;
            if (P.D3 == 3) {
                float* at = orow + (long long)(j0 / 3) * caps_out;
#pragma unroll
                for (int k = 0; k < RUNS; ++k)
                    if (j0 + 3 * k < P.cols) *reinterpret_cast<run_t*>(at + (long long)k * caps_out) = run_of(k);
            } else {
#pragma unroll
                for (int k = 0; k < RUNS; ++k) {
                    const int j = j0 + 3 * k;
                    const int m = (int)((unsigned)j / (unsigned)P.D3), d3 = j - m * P.D3;
                    if (j < P.cols) *reinterpret_cast<run_t*>(orow + (long long)m * caps_out + d3) = run_of(k);
                }
            }
        } else {
            // lane (h, lr) of tile (a, b) holds in registers 4g .. 4g+3 the columns 8g + 4h + 0..3 of
            // the tile for output row lr of the tile
            const bool st4 = (P.D3 & 3) == 0;
#pragma unroll
            for (int a = 0; a < TN; ++a) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int j0 = col0 + a * 32 + 8 * g + 4 * h;
                    if (st4) {
                        if (j0 < P.cols) {
                            const int m = (int)((unsigned)j0 / (unsigned)P.D3), d3 = j0 - m * P.D3;
                            const float4v v = {acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                                               acc[a][b][4 * g + 3]};
                            *reinterpret_cast<float4v*>(orow + (long long)m * caps_out + d3) = v;
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int j = j0 + u;
                            if (j < P.cols) {
                                // j / D3 by multiplication (exact while j * D3 < 2^32, which the host has checked)
                                const int m = P.d3_magic ? (int)__umulhi((unsigned)j, P.d3_magic) : j / P.D3;
                                const int d3 = j - m * P.D3;
                                orow[(long long)m * caps_out + d3] = acc[a][b][4 * g + u];
                            }
                        }
                    }
                }
            }
        }
    }
}

// Kernel repack: Kp[d0][column tile][K step][term of the split][half wave][column][8 bf16], in the
// K order the contraction walks.
struct SplitRepackParams {
    const float* kernel;
    chunk_t* kp;
    int ntaps, kw, D2, D3, KT, cols, bn, col_tiles, ksteps, nstages, cw;
    int triple, tile_cols;  // column order, see tile_columns
    long long k_base, k_sp, k_sq, k_sc, k_sm, k_sd0, k_sd2, k_sd3;
    unsigned total;  // threads
};
// One thread per pair of values, which share the stage and are neighbours in K: index arithmetic bounds this pass, and
// with a thread per 8 values (a set of divisions each, 64-bit ones for the place) the few waves of a kernel tensor
// ran it one after the other.  1.0 MB of kernel (32 -> 32 channels of 3x3x3, 3x3 window): 9.8 -> 6.1 us; a forward pass
// of it over 16 images of 16x16 59.2 -> 54.8, of 4x4 capsules 42.9 -> 39.5.
__global__ __launch_bounds__(256) void repack_split_kernel(const SplitRepackParams P)
{
    const unsigned id = blockIdx.x * 256 + threadIdx.x;
    if (id >= P.total) return;
    const unsigned pair = id & 3;
    unsigned r = id >> 2, next = r / (unsigned)P.bn;
    const int jl = (int)(r - next * (unsigned)P.bn);
    const int h = (int)(next & 1);
    r = next >> 1;
    const unsigned tile = r / (unsigned)P.ksteps;
    const int ks = (int)(r - tile * (unsigned)P.ksteps);
    const int d0 = (int)(tile / (unsigned)P.col_tiles), col_tile = (int)tile - d0 * P.col_tiles;
    // column of the tile at place jl of the matrix instructions' order
    int j = jl;
    if (P.triple) {
        const int hw = (jl >> 2) & 1, reg = jl / 32 * 16 + (jl & 31) / 8 * 4 + (jl & 3);
        j = reg < P.tile_cols / 2 ? hw * (P.tile_cols / 2) + reg : P.cols;  // (past the last run: none)
    }
    j += col_tile * P.tile_cols;
    // stage, and first value of the pair among those of the half wave's 2 slots, that the contraction has here
    unsigned stage = (unsigned)ks, v = 2 * pair;
    if (P.cw == 3) {
        const unsigned dword = 4 * (stage % 3) + pair, quarter = dword / 3;
        stage = stage / 3 * 4 + quarter;
        v = 2 * (dword - 3 * quarter);
    }
    const unsigned grp = stage / (unsigned)P.ntaps, tap = stage - grp * (unsigned)P.ntaps;
    const int k = ((int)grp * SLOTS + 2 * h) * P.cw + (int)v;
    float x[2] = {0.f, 0.f};
    if ((int)stage < P.nstages && k < P.KT && j < P.cols) {
        const int c = (int)((unsigned)k / (unsigned)P.D2), d2 = k - c * P.D2;
        const int p = (int)(tap / (unsigned)P.kw), q = (int)tap - p * P.kw;
        const int m = (int)((unsigned)j / (unsigned)P.D3), d3 = j - m * P.D3;
        const float* src = P.kernel + (P.k_base + p * P.k_sp + q * P.k_sq + c * P.k_sc + m * P.k_sm + d0 * P.k_sd0 +
                                       d2 * P.k_sd2 + d3 * P.k_sd3);
        x[0] = *src;
        if (k + 1 < P.KT) x[1] = src[d2 + 1 < P.D2 ? P.k_sd2 : P.k_sc - d2 * P.k_sd2];
    }
    unsigned short t[2][3];
    split_kernel_value(x[0], t[0]);
    split_kernel_value(x[1], t[1]);
    const size_t step = (size_t)tile * P.ksteps + ks;
    unsigned* kp = reinterpret_cast<unsigned*>(P.kp);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        kp[(((step * 3 + i) * 2 + h) * P.bn + jl) * 4 + pair] = t[0][i] | (unsigned)t[1][i] << 16;
}

template <int CW, int TN, int NW, bool TRIPLE>
hipError_t launch_one(const Dma32Params& P, long long blocks, hipStream_t stream)
{
    auto kern = igemm32_split_kernel<CW, TN, NW, TRIPLE>;
    const size_t lds_bytes = (size_t)(NBA * SLOTS * 64 * NW + kernel_ring(TN) * 6 * 32 * TN) * 16;
    static std::atomic<unsigned long long> lds_set{0};
    hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), (int)lds_bytes, lds_set);
    if (err != hipSuccess) return err;
    kern<<<dim3((unsigned)blocks), dim3(64 * NW), lds_bytes, stream>>>(P);
    return hipGetLastError();
}

template <int CW, int NW, bool TRIPLE>
hipError_t launch_tn(const Dma32Params& P, int tn, long long blocks, hipStream_t stream)
{
    switch (tn) {
        case 1: return launch_one<CW, 1, NW, TRIPLE>(P, blocks, stream);
        case 2: return launch_one<CW, 2, NW, TRIPLE>(P, blocks, stream);
        case 3: return launch_one<CW, 3, NW, TRIPLE>(P, blocks, stream);
        default: return launch_one<CW, 4, NW, TRIPLE>(P, blocks, stream);
    }
}

template <int NW, bool TRIPLE>
hipError_t launch_cw(const Dma32Plan& pl, hipStream_t stream)
{
    return pl.cw == 3 ? launch_tn<3, NW, TRIPLE>(pl.P, pl.tn, pl.blocks, stream)
                      : launch_tn<4, NW, TRIPLE>(pl.P, pl.tn, pl.blocks, stream);
}

bool triple_columns(int D3) { return D3 % 3 == 0 && D3 % 4 != 0; }

}  // namespace

int igemm32_split_period(int cw) { return stage_period(cw); }
// bf16 matrix instruction steps (16 K values) of a K loop of `stages` stages, whole periods
int igemm32_split_ksteps(int cw, int stages) { return cw == 3 ? (stages + 3) / 4 * 3 : (stages + 1) / 2 * 2; }

int igemm32_split_tile_columns(int D3, int tn) { return tile_columns(triple_columns(D3), tn); }

hipError_t launch_igemm32_split(const Dma32Plan& pl, hipStream_t stream)
{
    if (triple_columns(pl.P.D3))
        return pl.nw == 4 ? launch_cw<4, true>(pl, stream) : launch_cw<1, true>(pl, stream);
    return pl.nw == 4 ? launch_cw<4, false>(pl, stream) : launch_cw<1, false>(pl, stream);
}

hipError_t launch_repack_split(const ConvShape& s, const Dma32Plan& pl, const void* kernel, void* kp,
                               hipStream_t stream)
{
    SplitRepackParams R;
    R.kernel = static_cast<const float*>(kernel);
    R.kp = static_cast<chunk_t*>(kp);
    R.ntaps = pl.P.ntaps; R.kw = s.kw; R.D2 = s.D2; R.D3 = s.D3; R.KT = s.C * s.D2;
    R.cols = pl.P.cols; R.bn = 32 * pl.tn; R.col_tiles = pl.P.col_tiles; R.ksteps = pl.P.ksteps;
    R.nstages = pl.P.nstages; R.cw = pl.cw;
    R.triple = triple_columns(s.D3);
    R.tile_cols = igemm32_split_tile_columns(s.D3, pl.tn);
    if (s.kernel_view) {
        R.k_base = s.k_base; R.k_sp = s.k_sp; R.k_sq = s.k_sq; R.k_sc = s.k_sc;
        R.k_sm = s.k_sm; R.k_sd0 = s.k_sd0; R.k_sd2 = s.k_sd2; R.k_sd3 = s.k_sd3;
    } else {  // dense [kh][kw][C][M][D0][D2][D3]
        R.k_base = 0;
        R.k_sd3 = 1;
        R.k_sd2 = s.D3;
        R.k_sd0 = (long long)s.D2 * s.D3;
        R.k_sm = R.k_sd0 * s.D0;
        R.k_sc = R.k_sm * s.M;
        R.k_sq = R.k_sc * s.C;
        R.k_sp = R.k_sq * s.kw;
    }
    R.total = (unsigned)(pl.repack_bytes / 12);  // (igemm32_dma_eligible keeps the packed kernel below 2 GiB)
    repack_split_kernel<<<(R.total + 255) / 256, 256, 0, stream>>>(R);
    return hipGetLastError();
}

}  // namespace capscaps
