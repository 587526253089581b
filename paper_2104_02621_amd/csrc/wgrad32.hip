// Kernel gradient of the capsule convolution for fp32 operands on the matrix cores: one GEMM per
// window tap (rows (c,d2), columns (m,d3), K = (n,x,y,d1) over the output pixels whose tap lies
// inside the image; the K_diff result of the paper's Algorithm 4 read as the derivative of
// Algorithm 2's sum), for capsule heights D1 of 3, 4, 6, 8, 12 or 16 floats.
//
// Bound: the matrix rate.  As in igemm32_split.hip every fp32 value, times 2^23, is the exact sum of
// three bf16 values (bf16_split.h) and six bf16 products take the place of one fp32 product: 192
// instead of 512 cycles per 32 x 32 tile and 16 K values; a workgroup with a sum that is not finite
// takes its sums again on the fp32 instructions.  Both operands are split in
// registers, so the tile is what decides: a workgroup is ONE wave with up to 96 x 96 of the result
// (3 x 3 MFMA tiles: 54 matrix instructions beside 216 vector instructions of splitting per 16 K
// values), with LDS of its own and no barrier.  Measured (N = 64, 32x32, 3x3, 32 -> 32 channels of
// 3x3x3 capsules): 0.92 ms on the fp32 instructions with 128 x 96 tiles of two waves, 0.66 ms here
// (error against 64-bit sums 1.05e-6 and 7.8e-7); 35 % of the cycles issue no matrix instruction
// for LDS reads of single floats with bank conflicts, the splitting and the pixel walk of one wave.
//
// fp32 layers have few rows and columns per tap (32 channels of 3x3x3 capsules: 96 x 96) and a very
// long K, so the K loop -- every tap's sequence of valid output pixels -- is cut into equal ranges
// over the waves of the chip (partial sums to scratch, added in a fixed order by the shared
// reduction kernel).
//
// Unless the capsules are square (see NAT below), a pre-pass writes capsule-transposed copies
// It[n][h][w][c][d0][d2][d1] and Gt[n][x][y][m][d0][d3][d1], so the D1 contracted values of one
// (pixel, row) are contiguous.
// Data moves in 16-byte LDS slots of CW = 3 or 4 floats ("chunks", D1 = CW * D1C): a 12-byte
// buffer load lands at a 16-byte lane stride in LDS.  A stage is 4 slots of every row and column
// = 4/D1C pixels; the lower half wave takes the first half of the stage's K values, the upper the
// second: 8 values (CW = 4), the K extent of one bf16 instruction, or 6 (CW = 3), so that four
// stages make three instructions' worth.  A stage's values are read from LDS and split one stage
// ahead of their use, between the matrix instructions of the stage before.
#include <hip/hip_runtime.h>

#include <cmath>

#include "bf16_split.h"
#include "igemm_common.h"
#include "lds_dma.h"

namespace capscaps {
namespace {

constexpr int SLOTS = 4;  // per row or column and stage
// stages the K loop's body covers (as in igemm32_split.hip)
constexpr int stage_period(int cw) { return cw == 3 ? 4 : 2; }
// Ring of LDS stages: three, or two where that lets eight waves share a CU (64 x 64 tiles: 16 KB).
constexpr int ring_depth(int tm, int tn) { return tm == 2 && tn == 2 ? 2 : 3; }
constexpr int lds_bytes_of(int tm, int tn) { return ring_depth(tm, tn) * SLOTS * 32 * (tm + tn) * 16; }

struct Wgrad32Params {
    const void* it;  // capsule-transposed input, or the input itself
    const void* gt;  // capsule-transposed output gradient, or the output gradient itself
    float* out;      // dK, or partial sums [split][kernel elements]
    int N, H, W, C, M, kw, stride, pad, D0, D1, D2, D3, Ho, Wo;
    int D1C;         // chunks per capsule column: D1 = CW * D1C, D1C in {1, 2, 4}
    int rows, cols;  // C*D2, M*D3
    int row_step, col_step;  // rows and columns of a tile
    int row_tiles, col_tiles, ntaps;
    int tiles;       // ntaps * D0 * row_tiles * col_tiles
    int natural;          // 1: it / gt are the input and the output gradient themselves
    unsigned d3_magic;    // ceil(2^32 / D3): column index / D3 as a multiplication; 0 = divide
    int nsplit;           // ranges the K loop (a tap's valid output pixels) is cut into
    long long items;      // tiles * nsplit = workgroups
    long long out_elems;  // elements of dK
    long long it_img_bytes, gt_img_bytes;
};

// What a workgroup contracts: a tile of a tap's products over a range of the tap's pixels.
struct Item {
    int split, row_tile, col_tile, tap, d0, tp, tq;
    // Per image the output pixels whose tap (tp, tq) reads a real input pixel form a rectangle of nx x ny
    // from (x_lo, y_lo) on; the rectangles of all images, image after image, row after row, are one
    // sequence, cut into nsplit equal ranges.  This one's has npix pixels, from (xs, ys) of the
    // rectangle of image n0 to image n_last.
    int nx, ny, x_lo, y_lo, npix, n0, n_last, xs, ys;
    __device__ __forceinline__ explicit Item(const Wgrad32Params& P)
    {
        // each XCD (workgroups are dealt to the 8 XCDs in turn) gets a contiguous range of items,
        // pixel range slowest, so its resident workgroups read the same pixels
        long long item = blockIdx.x;
        const long long per = P.items / 8;
        if (item < per * 8) item = (item % 8) * per + item / 8;
        split = (int)(item / P.tiles);
        int rest = (int)(item % P.tiles);
        col_tile = rest % P.col_tiles;
        rest /= P.col_tiles;
        row_tile = rest % P.row_tiles;
        rest /= P.row_tiles;
        tap = rest % P.ntaps;
        d0 = rest / P.ntaps;
        tp = tap / P.kw;
        tq = tap - tp * P.kw;
        const int s = P.stride;
        const int tx = P.pad - tp, ty = P.pad - tq;
        x_lo = tx > 0 ? (tx + s - 1) / s : 0;
        y_lo = ty > 0 ? (ty + s - 1) / s : 0;
        const int hx = P.H - 1 + tx, hy = P.W - 1 + ty;
        int x_hi = hx >= 0 ? hx / s : -1, y_hi = hy >= 0 ? hy / s : -1;
        if (x_hi > P.Ho - 1) x_hi = P.Ho - 1;
        if (y_hi > P.Wo - 1) y_hi = P.Wo - 1;
        nx = x_hi - x_lo + 1;
        ny = y_hi - y_lo + 1;
        if (nx <= 0 || ny <= 0) nx = ny = 0;
        const long long rect = (long long)nx * ny, total = rect * P.N;
        const long long tps = (total + P.nsplit - 1) / P.nsplit;
        long long t0 = (long long)split * tps;
        if (t0 > total) t0 = total;
        long long t1 = t0 + tps;
        if (t1 > total) t1 = total;
        npix = (int)(t1 - t0);
        n0 = npix > 0 ? (int)(t0 / rect) : 0;
        n_last = npix > 0 ? (int)((t1 - 1) / rect) : n0;
        const int r0 = npix > 0 ? (int)(t0 - (long long)n0 * rect) : 0;  // position in image n0
        xs = ny > 0 ? r0 / ny : 0;
        ys = ny > 0 ? r0 - xs * ny : 0;
    }
};

// dst[x][b][a] = src[x][a][b] for matrices of A x B floats.  One thread per 4 neighbours of dst (on a 16-byte boundary).
// Index arithmetic bounds it, not the two passes over memory: one set of divisions per 4 values, 32-bit ones where the
// count fits (I).  Against a thread and two 64-bit divisions per value, the whole call: 20 images of 31x27, 20 -> 14
// channels of 6x5 . 5x4, 5x5 window, trained, 736 -> 715 us; both gradients of 32 images of 20x20, 32 -> 24 channels of
// 4x8 . 8x4, 346 -> 325.
template <typename I>
__global__ __launch_bounds__(256) void transpose_caps32_kernel(const float* __restrict__ src,
                                                               float* __restrict__ dst, int A,
                                                               int B, I total)
{
    const I id = ((I)blockIdx.x * 256 + threadIdx.x) * 4;
    if (id >= total) return;
    const I rest = id / (I)A, mat = rest / (I)B;
    int a = (int)(id - rest * (I)A), b = (int)(rest - mat * (I)B);
    const float* p = src + (size_t)mat * A * B;
    const int n = total - id < 4 ? (int)(total - id) : 4;
    float4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (e < n) v[e] = p[a * B + b];
        if (++a == A) {
            a = 0;
            if (++b == B) {
                b = 0;
                p += A * B;
            }
        }
    }
    if (n == 4) {
        *reinterpret_cast<float4v*>(dst + id) = v;
    } else {
        for (int e = 0; e < n; ++e) dst[id + e] = v[e];
    }
}

// NAT = 0: the operands are the capsule-transposed copies.  NAT = 1 (one chunk per capsule column)
// or 2 (two or four): they are the tensors themselves (square capsules, D1 = D2 = D3).  The copies are the same -- lane i then brings row
// (c, d1) with its d2 values where the transposed tensor has row (c, d2) with its d1 values, at the
// same byte offsets -- and the values are picked out of the slots one by one: row (c, d2) at K
// index (pixel, d1) is element d2 of slot (pixel, c, d1).
template <int CW, int TM, int TN, int NAT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(TM + TN <= 4 ? 2 : 1)))
void wgrad32_kernel(const Wgrad32Params P)
{
    constexpr int PER = stage_period(CW), NB = ring_depth(TM, TN);
    constexpr int RA = 32 * TM, RB = 32 * TN, TT = TM + TN;
    constexpr int A_BYTES = SLOTS * RA * 16, B_BYTES = SLOTS * RB * 16, STAGE_BYTES = A_BYTES + B_BYTES;
    constexpr int GA = (RA + 63) / 64, GB = (RB + 63) / 64;  // copies per slot
    constexpr int NCOPY = SLOTS * (GA + GB);                 // ... per stage
    constexpr int NPAIR = TT * CW;                           // pairs of values to split per stage
    constexpr int WORDS = PER * CW;                          // pairs per tile and period
    constexpr int OOB = (int)0x80000000u;
    constexpr int NO_PIXEL = 0x7fffff00;  // no tensor range here is that long
    constexpr int KEEP = (NB - 2) * NCOPY;  // copies that may be in flight when a stage begins
    static_assert(KEEP < 64, "vmcnt is a 6-bit counter");
    constexpr int VMCNT_KEEP = 0x0F70 | (KEEP & 15) | ((KEEP >> 4) << 14);

    extern __shared__ char smem[];

    // ---- the item, and its pixels
    const Item it(P);
    const int split = it.split, row_tile = it.row_tile, col_tile = it.col_tile, tap = it.tap, d0 = it.d0;
    const int tp = it.tp, tq = it.tq, nx = it.nx, ny = it.ny, x_lo = it.x_lo, y_lo = it.y_lo;
    const int npix = it.npix, n0 = it.n0, n_last = it.n_last, xs = it.xs, ys = it.ys, s = P.stride;

    const int lane = threadIdx.x & 63;
    const int h = lane >> 5, lr = lane & 31;
    const int ipix = P.C * P.D0 * P.D2 * P.D1 * 4;  // bytes per pixel of It / Gt
    const int gpix = P.M * P.D0 * P.D3 * P.D1 * 4;
    const int i_step = s * ipix, g_step = gpix;
    const int i_rowjump = (s * P.W - (ny - 1) * s) * ipix, g_rowjump = (P.Wo - (ny - 1)) * gpix;
    const int i_imgjump = (P.H * P.W - nx * s * P.W) * ipix, g_imgjump = (P.Ho * P.Wo - nx * P.Wo) * gpix;
    // offsets are relative to image n0
    const int i_begin = (((x_lo + xs) * s - (P.pad - tp)) * P.W + ((y_lo + ys) * s - (P.pad - tq))) * ipix;
    const int g_begin = ((x_lo + xs) * P.Wo + y_lo + ys) * gpix;
    const int n1 = n_last + 1;

    const char* it_base = static_cast<const char*>(P.it) + (long long)n0 * P.it_img_bytes;
    const char* gt_base = static_cast<const char*>(P.gt) + (long long)n0 * P.gt_img_bytes;
    const rsrc_t rs_it = make_rsrc(it_base, (unsigned)((n1 - n0) * P.it_img_bytes));
    const rsrc_t rs_gt = make_rsrc(gt_base, (unsigned)((n1 - n0) * P.gt_img_bytes));
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;

    // ---- per-lane constants: byte offset of the lane's row (column) within a pixel, or the
    // out-of-range mark past the last row (column) of the tile: those copy zeros
    unsigned a_voff[GA], b_voff[GB];
#pragma unroll
    for (int u = 0; u < GA; ++u) {
        const int rl = 64 * u + lane, R = row_tile * P.row_step + rl;
        const int c = R / P.D2, d2 = R - c * P.D2;
        a_voff[u] = rl < P.row_step && R < P.rows ? (unsigned)((((c * P.D0 + d0) * P.D2 + d2) * P.D1) * 4)
                                                  : (unsigned)OOB;
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const int jl = 64 * u + lane, J = col_tile * P.col_step + jl;
        const int m = J / P.D3, d3 = J - m * P.D3;
        b_voff[u] = jl < P.col_step && J < P.cols ? (unsigned)((((m * P.D0 + d0) * P.D3 + d3) * P.D1) * 4)
                                                  : (unsigned)OOB;
    }
    const int pps = NAT == 1 ? SLOTS : SLOTS / P.D1C;  // pixels per stage
    const int nstages = (npix + pps - 1) / pps;

    // Scalar pixel walk: a stage's pixels, each the next valid output pixel of the tap's rectangle,
    // image after image; past the last one the out-of-range mark NO_PIXEL, which stays out of range
    // without wrapping around when a lane's mark and a chunk's offset are added to it.  Three pieces
    // of scalar instructions, written out: from C++ the compiler makes four times as many.
    int left, yl, xl, i_cur, g_cur;
    int i_soff[SLOTS], g_soff[SLOTS];
    auto restart = [&]() {
        left = npix;
        yl = ny - ys;
        xl = nx - xs;
        i_cur = i_begin;
        g_cur = g_begin;
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) i_soff[j] = g_soff[j] = NO_PIXEL;
    };
    int i_add, g_add, row_done;
    auto walk = [&](int j, int piece) {
        if (piece == 0) {
            asm volatile("s_cmp_gt_i32 %2, 0\n\ts_cselect_b32 %0, %3, %5\n\ts_cselect_b32 %1, %4, %5\n\t"
                         "s_sub_i32 %2, %2, 1"
                         : "=&s"(i_soff[j]), "=&s"(g_soff[j]), "+s"(left)
                         : "s"(i_cur), "s"(g_cur), "s"(NO_PIXEL) : "scc");
        } else if (piece == 1) {
            asm volatile("s_sub_i32 %0, %0, 1\n\ts_cmp_eq_u32 %0, 0\n\ts_cselect_b32 %1, %4, %5\n\t"
                         "s_cselect_b32 %2, %6, %7\n\ts_cselect_b32 %0, %8, %0\n\ts_cselect_b32 %3, 1, 0"
                         : "+s"(yl), "=&s"(i_add), "=&s"(g_add), "=&s"(row_done)
                         : "s"(i_rowjump), "s"(i_step), "s"(g_rowjump), "s"(g_step), "s"(ny) : "scc");
            asm volatile("s_add_i32 %0, %0, %3\n\ts_add_i32 %1, %1, %4\n\ts_sub_i32 %2, %2, %5"
                         : "+s"(i_cur), "+s"(g_cur), "+s"(xl) : "s"(i_add), "s"(g_add), "s"(row_done) : "scc");
        } else {
            asm volatile("s_cmp_eq_u32 %0, 0\n\ts_cselect_b32 %1, %5, 0\n\ts_cselect_b32 %2, %6, 0\n\t"
                         "s_cselect_b32 %0, %7, %0\n\ts_add_i32 %3, %3, %1\n\ts_add_i32 %4, %4, %2"
                         : "+s"(xl), "=&s"(i_add), "=&s"(g_add), "+s"(i_cur), "+s"(g_cur)
                         : "s"(i_imgjump), "s"(g_imgjump), "s"(nx) : "scc");
        }
    };
    constexpr int PIECES = 3;
    auto walk_stage = [&]() {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j)
            if (j < pps)
#pragma unroll
                for (int k = 0; k < PIECES; ++k) walk(j, k);
    };
    // copy c (0 .. NCOPY-1) of the stage whose pixels have been walked, into the ring slot at `stage`
    auto copy = [&](unsigned stage, auto C_) {
        constexpr int c = decltype(C_)::value, q = c / (GA + GB), u = c % (GA + GB);
        constexpr bool is_a = u < GA;
        constexpr int g = is_a ? u : u - GA, R = is_a ? RA : RB;
        constexpr bool half = 64 * g + 64 > R;  // the last 32 rows
        const int(&soff)[SLOTS] = is_a ? i_soff : g_soff;
        int so = soff[q];
        if constexpr (NAT != 1) {  // slots of one pixel: its consecutive chunks
            so = P.D1C == 1 ? so : P.D1C == 2 ? soff[q / 2] + (q % 2) * CW * 4 : soff[0] + q * CW * 4;
        }
        copy_to_lds_at<CW, half, (is_a ? 0 : A_BYTES) + (q * R + 64 * g) * 16>(
            is_a ? rs_it : rs_gt, stage, is_a ? a_voff[g < GA ? g : 0] : b_voff[g < GB ? g : 0], so);
    };

    float16v acc[TN][TM];
    auto clear_acc = [&]() {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    };

    // ---- LDS offsets of this lane's values: tiles 0 .. TM-1 are row tiles, TM .. column tiles
    unsigned rd[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        const int R = t < TM ? RA : RB, base = t < TM ? 0 : A_BYTES;
        const int rl = 32 * (t < TM ? t : t - TM) + lr;
        if constexpr (NAT) {
            const int D = P.D2;  // = D1 = D3
            const bool real = t < TM ? rl < P.row_step && row_tile * P.row_step + rl < P.rows
                                     : rl < P.col_step && col_tile * P.col_step + rl < P.cols;
            const int c_l = real ? rl / D : 0, d = real ? rl - c_l * D : 0;
            // the half wave's first K index is (pixel, d1) = (2h, 0), (h, 0) or (0, 2 CW h)
            const int k0 = NAT == 1 || P.D1C == 2 ? 2 * h * R : 2 * CW * h;
            rd[t] = (unsigned)(base + (k0 + (d / CW) * R + c_l * D) * 16 + (d % CW) * 4);
        } else {
            rd[t] = (unsigned)(base + (2 * h * R + rl) * 16);
        }
    }
    // value v (0 .. 2 CW - 1) of tile t of the stage at `slot`
    auto read_one = [&](const char* slot, int t, int v) -> float {
        const int R = t < TM ? RA : RB;
        const int off = NAT == 1 ? (v / CW) * R + v % CW : v;
        return *reinterpret_cast<const float*>(slot + rd[t] + off * 16);
    };
    auto read_chunk = [&](const char* slot, int t, int u) -> float4v {
        return *reinterpret_cast<const float4v*>(slot + rd[t] + u * (t < TM ? RA : RB) * 16);
    };
    // all values of a tile, as pairs
    auto take_tile = [&](const char* slot, int t, float* lo, float* hi) {
        if constexpr (NAT) {
#pragma unroll
            for (int i = 0; i < CW; ++i) {
                lo[i] = read_one(slot, t, 2 * i);
                hi[i] = read_one(slot, t, 2 * i + 1);
            }
        } else {
            const float4v raw[2] = {read_chunk(slot, t, 0), read_chunk(slot, t, 1)};
#pragma unroll
            for (int i = 0; i < CW; ++i) {
                lo[i] = raw[2 * i / CW][2 * i % CW];
                hi[i] = raw[(2 * i + 1) / CW][(2 * i + 1) % CW];
            }
        }
    };

    // ---- the K loop on the split values
    {
        const MinusOne one;
        unsigned iv[TT][3][WORDS];   // split values of one period: pairs per tile and term
        float lo[NPAIR], hi[NPAIR];  // the pairs being split: what the terms so far leave over
        // The bf16 instructions drop what lies far below the accumulator's last bit toward minus
        // infinity: 2^-9 of that bit on average, but always the same way, which over the long K of
        // a kernel gradient adds up (K = 262144: to more than all the rounding).  So the sums are
        // taken with alternating sign: every FLIP stages the accumulators and the row operand
        // change sign, every other range begins with the other sign, and the dropped parts cancel.
        constexpr int FLIP = 48;  // a multiple of both periods
        unsigned row_scale = __builtin_bit_cast(unsigned, SPLIT_SCALE) | (unsigned)split << 31;  // of the row values being split
        // step `k` (0 .. SPLIT_STEPS - 1) of splitting pair `p` of a stage at place `pos` of the period
        auto split_step = [&](int p, int k, int pos) {
            unsigned(&w)[3][WORDS] = iv[p / CW];
            const int at = pos * CW + p % CW, t = (k - 2) / 3;
            const float scale = p / CW < TM ? __builtin_bit_cast(float, row_scale) : SPLIT_SCALE;
            if (k == 0) {
                lo[p] *= scale;
                asm volatile("" : "+v"(lo[p]));  // (stays in the gap it is dealt to)
            } else if (k == 1) {
                hi[p] *= scale;
                asm volatile("" : "+v"(hi[p]));
            } else if (k % 3 == 2) {
                w[t][at] = round_pair(lo[p], hi[p]);
                asm volatile("" : "+v"(w[t][at]));
            } else if (k % 3 == 0) {
                lo[p] = minus_bf16(lo[p], w[t][at], one.lo);
                asm volatile("" : "+v"(lo[p]));
            } else {
                hi[p] = minus_bf16(hi[p], w[t][at], one.hi);
                asm volatile("" : "+v"(hi[p]));
            }
        };
        // matrix instruction n of a period (stays in its place, like the splitting)
        auto multiply = [&](auto N_) {
            constexpr int n = decltype(N_)::value, NM = TN * TM * SPLIT_PRODUCTS;
            constexpr int i = n % NM, W0 = n / NM * 4;  // (W0: the K step's first pair)
            constexpr int b = i % TM, a = i / TM % TN, u = i / (TM * TN);
            const unsigned(&wk)[WORDS] = iv[TM + a][SPLIT_TERM_A[u]];
            const unsigned(&wi)[WORDS] = iv[b][SPLIT_TERM_B[u]];
            const chunk_t kf = {wk[W0], wk[W0 + 1], wk[W0 + 2], wk[W0 + 3]};
            const chunk_t xf = {wi[W0], wi[W0 + 1], wi[W0 + 2], wi[W0 + 3]};
            asm volatile("" : "+a"(acc[a][b]));
            Mma<bf16_tag>::run(kf, xf, acc[a][b]);
            asm volatile("" : "+a"(acc[a][b]));
        };
        if constexpr (CW == 3) {  // the first period's first stage multiplies zeros
#pragma unroll
            for (int t = 0; t < TT; ++t)
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int i = 8; i < 12; ++i) iv[t][k][i] = 0;
        }
        clear_acc();
        restart();
        // prologue: NB stages in flight, the first landed, read and split; its slot is free then
        static_for<NB>([&](auto S0) {
            walk_stage();
            static_for<NCOPY>([&](auto C_) { copy(lds0 + decltype(S0)::value * STAGE_BYTES, C_); });
        });
        {
            constexpr int keep0 = (NB - 1) * NCOPY;
            static_assert(keep0 < 64, "vmcnt is a 6-bit counter");
            __builtin_amdgcn_s_waitcnt(0x0F70 | (keep0 & 15) | ((keep0 >> 4) << 14));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < TT; ++t) take_tile(smem, t, lo + t * CW, hi + t * CW);
#pragma unroll
        for (int k = 0; k < SPLIT_STEPS; ++k)
#pragma unroll
            for (int p = 0; p < NPAIR; ++p) split_step(p, k, 0);
        __builtin_amdgcn_s_waitcnt(VMCNT_KEEP & 0xF0FF);  // stage 1 has landed, the reads are done
        asm volatile("" ::: "memory");
        unsigned cur = 0;  // ring slot of this stage: free, takes the stage NB ahead
        int to_flip = FLIP;
        for (int st = 0; st < nstages; st += PER) {
            if (to_flip == 0) {
                to_flip = FLIP;
                row_scale ^= 0x80000000u;
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b) acc[a][b] = -acc[a][b];
                // the row values of the stage at hand are split already (CW = 3: as are those of the
                // K step at hand)
#pragma unroll
                for (int b = 0; b < TM; ++b)
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int i = 0; i < WORDS; ++i)
                            if (i < CW || (CW == 3 && i >= 8)) iv[b][t][i] ^= 0x80008000u;
            }
            to_flip -= PER;
            static_for<PER>([&](auto POS) {
                constexpr int pos = decltype(POS)::value, next = (pos + 1) % PER;
                // matrix instructions [first, last) of the period's: those of one K step (CW = 4), or
                // a quarter of three K steps', which begin when the second stage is split and end
                // in the next period's first stage
                constexpr int NM = TN * TM * SPLIT_PRODUCTS, quarter = (pos + 3) % 4;
                constexpr int first = CW == 4 ? pos * NM : quarter * 3 * NM / 4;
                constexpr int last = CW == 4 ? first + NM : (quarter + 1) * 3 * NM / 4;
                constexpr int NMMA = last - first;
                const unsigned nxt = cur + STAGE_BYTES == NB * STAGE_BYTES ? 0 : cur + STAGE_BYTES;
#pragma unroll
                for (int t = 0; t < TT; ++t) take_tile(smem + nxt, t, lo + t * CW, hi + t * CW);
                // side operations, dealt out over the gaps after the matrix instructions: the
                // pixel walk and the copies of the stage NB ahead, the next stage's splitting
                constexpr int NSTEP = SPLIT_STEPS * NPAIR, GAPS = NMMA;
                constexpr int FIRST = NMMA / 6;  // the values need time to arrive
                constexpr int NWALK = SLOTS * PIECES, NSIDE = NWALK + NCOPY;
                static_for<GAPS>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    multiply(std::integral_constant<int, first + i>{});
                    constexpr int j0 = dealt_before(i, NSIDE, GAPS, 0), j1 = dealt_before(i + 1, NSIDE, GAPS, 0);
                    static_for<j1 - j0>([&](auto J) {
                        constexpr int j = j0 + decltype(J)::value;
                        if constexpr (j < NWALK) {
                            if (j / PIECES < pps) walk(j / PIECES, j % PIECES);
                        } else {
                            copy(lds0 + cur, std::integral_constant<int, j < NWALK ? 0 : j - NWALK>{});
                        }
                    });
                    constexpr int t0 = dealt_before(i, NSTEP, GAPS, FIRST), t1 = dealt_before(i + 1, NSTEP, GAPS, FIRST);
#pragma unroll
                    for (int t = t0; t < t1; ++t) split_step(t % NPAIR, t / NPAIR, next);
                    __builtin_amdgcn_sched_barrier(0);
                });
                // the copies of the stage after the next have landed, the reads are done
                __builtin_amdgcn_s_waitcnt(VMCNT_KEEP & 0xF0FF);
                asm volatile("" ::: "memory");
                cur = nxt;
            });
        }
        // the copies of the surplus stages still write (zeros) into this workgroup's LDS
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if constexpr (CW == 3) {  // the last period's last quarter
            constexpr int NM3 = 3 * TN * TM * SPLIT_PRODUCTS, begin = 3 * NM3 / 4;
            static_for<NM3 - begin>([&](auto I) { multiply(std::integral_constant<int, begin + decltype(I)::value>{}); });
        }
        const float unscale = row_scale >> 31 ? -SPLIT_UNSCALE : SPLIT_UNSCALE;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) acc[a][b] *= unscale;
    }

    // ---- the same sums on the fp32 matrix instructions, one stage at a time
    auto contract_exact = [&]() {
        clear_acc();
        restart();
        for (int st = 0; st < nstages; ++st) {
            walk_stage();
            static_for<NCOPY>([&](auto C_) { copy(lds0, C_); });
            __builtin_amdgcn_s_waitcnt(0x0F70);
            asm volatile("" ::: "memory");
            float lo[NPAIR], hi[NPAIR];
#pragma unroll
            for (int t = 0; t < TT; ++t) take_tile(smem, t, lo + t * CW, hi + t * CW);
#pragma unroll
            for (int i = 0; i < CW; ++i)
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b) {
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(lo[(TM + a) * CW + i], lo[b * CW + i], acc[a][b], 0, 0, 0);
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(hi[(TM + a) * CW + i], hi[b * CW + i], acc[a][b], 0, 0, 0);
                    }
            __builtin_amdgcn_s_waitcnt(0xC07F);
            asm volatile("" ::: "memory");
        }
    };
    {
        SplitCheck check;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) check.take(acc[a][b]);
        if (__builtin_amdgcn_ballot_w64(check.failed()) != 0) contract_exact();
    }

    // ---- epilogue: lane (h, lr) of tile (a, b) holds in registers 4g..4g+3 the columns
    // 8g + 4h + 0..3 of the tile for row lr of the tile
    float* __restrict__ out = P.out + (long long)split * P.out_elems;
    const long long caps = (long long)P.D0 * P.D2 * P.D3;
    const bool st4 = (P.D3 & 3) == 0;
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const int rl = b * 32 + lr, R = row_tile * P.row_step + rl;
        if (rl >= P.row_step || R >= P.rows) continue;
        const int c = R / P.D2, d2 = R - c * P.D2;
        float* orow = out + ((long long)tap * P.C + c) * P.M * caps +
                      ((long long)d0 * P.D2 + d2) * P.D3;
#pragma unroll
        for (int a = 0; a < TN; ++a) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int jl = a * 32 + 8 * g + 4 * h, j0 = col_tile * P.col_step + jl;
                if (st4) {
                    if (jl < P.col_step && j0 < P.cols) {
                        const int m = j0 / P.D3, d3 = j0 - m * P.D3;
                        float4v v = {acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                                     acc[a][b][4 * g + 3]};
                        *reinterpret_cast<float4v*>(orow + (long long)m * caps + d3) = v;
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = j0 + u;
                        if (jl + u < P.col_step && j < P.cols) {
                            // j / D3 by multiplication (exact while j * D3 < 2^32, which the host has checked)
                            const int m = P.d3_magic ? (int)__umulhi((unsigned)j, P.d3_magic) : j / P.D3;
                            const int d3 = j - m * P.D3;
                            orow[(long long)m * caps + d3] = acc[a][b][4 * g + u];
                        }
                    }
                }
            }
        }
    }
}

// The same contraction on the fp32 matrix instructions, for layers with at most 32 columns whose operands
// are transposed copies.  There the splitting does not pay: a wave of the kernel above takes two row tiles
// and one column tile, 1.5 splits per six products, and copies 3 KB to LDS per 32 x 32 results and 16 K
// values; here NW = 2 or 4 waves share a column tile, 64 rows each, and 2.25 KB.  Measured: 16 -> 8
// channels of 4x16 . 16x4 capsules, 25 images of 28x28, 6x6 window, stride 2: 147 us above, 131 here;
// 40 -> 8 channels of 6x5 . 5x4, 7 images of 36x20, 6x6: 164 and 133.  KCH chunks per row and stage, ring
// of three stages, one barrier per stage.
constexpr int NARROW_RING = 3;
constexpr int narrow_chunks(int d1c, int nw) { return d1c == 4 || nw == 4 ? 4 : 2; }
constexpr int narrow_lds_bytes(int nw, int kch) { return NARROW_RING * kch * (64 * nw + 64) * 16; }
template <int CW, int NW, int KCH>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(KCH == 2 ? 3 : 2)))
void wgrad32_narrow_kernel(const Wgrad32Params P)
{
    constexpr int NB = NARROW_RING, TM = 2;
    constexpr int BM = 64 * NW, BN = 64;  // (32 columns, copied by whole waves)
    constexpr int A_BYTES = KCH * BM * 16, B_BYTES = KCH * BN * 16, STAGE_BYTES = A_BYTES + B_BYTES;
    constexpr int BPW = KCH / NW;  // column-side copies per wave and stage
    static_assert(KCH % NW == 0, "column copies divide evenly over the waves");
    constexpr int KEEP = (NB - 2) * (KCH + BPW);  // copies that may be in flight at a barrier
    static_assert(KEEP < 16, "vmcnt's low bits");
    constexpr int OOB = (int)0x80000000u, NO_PIXEL = 0x7fffff00;  // (marks as in the kernel above)

    extern __shared__ char smem[];
    const Item it(P);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, lr = lane & 31;

    const int s = P.stride, ny = it.ny, nx = it.nx;
    const int ipix = P.C * P.D0 * P.D2 * P.D1 * 4, gpix = P.M * P.D0 * P.D3 * P.D1 * 4;
    const int i_step = s * ipix, g_step = gpix;
    const int i_rowjump = (s * P.W - (ny - 1) * s) * ipix, g_rowjump = (P.Wo - (ny - 1)) * gpix;
    const int i_imgjump = (P.H * P.W - nx * s * P.W) * ipix, g_imgjump = (P.Ho * P.Wo - nx * P.Wo) * gpix;
    int i_cur = (((it.x_lo + it.xs) * s - (P.pad - it.tp)) * P.W + ((it.y_lo + it.ys) * s - (P.pad - it.tq))) * ipix;
    int g_cur = ((it.x_lo + it.xs) * P.Wo + it.y_lo + it.ys) * gpix;
    int left = it.npix, yl = ny - it.ys, xl = nx - it.xs;
    const int images = it.n_last + 1 - it.n0;
    const rsrc_t rs_it = make_rsrc(static_cast<const char*>(P.it) + (long long)it.n0 * P.it_img_bytes,
                                   (unsigned)(images * P.it_img_bytes));
    const rsrc_t rs_gt = make_rsrc(static_cast<const char*>(P.gt) + (long long)it.n0 * P.gt_img_bytes,
                                   (unsigned)(images * P.gt_img_bytes));
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;

    unsigned a_voff, b_voff;
    {
        const int R = it.row_tile * BM + wave * 64 + lane, c = R / P.D2, d2 = R - c * P.D2;
        a_voff = R < P.rows ? (unsigned)((((c * P.D0 + it.d0) * P.D2 + d2) * P.D1) * 4) : (unsigned)OOB;
        const int m = lane / P.D3, d3 = lane - m * P.D3;
        b_voff = lane < P.cols ? (unsigned)((((m * P.D0 + it.d0) * P.D3 + d3) * P.D1) * 4) : (unsigned)OOB;
    }
    const int pps = KCH / P.D1C;  // pixels per stage
    const int d1c_shift = P.D1C == 1 ? 0 : P.D1C == 2 ? 1 : 2;
    const int nstages = (it.npix + pps - 1) / pps;

    // copies of the next stage, its pixels each the next valid output pixel of the tap's rectangle
    auto issue_stage = [&](int slot) {
        const unsigned stage = lds0 + slot * STAGE_BYTES;
        int i_soff[KCH], g_soff[KCH];
#pragma unroll
        for (int j = 0; j < KCH; ++j) {
            i_soff[j] = g_soff[j] = NO_PIXEL;
            if (j < pps) {
                if (left > 0) {
                    i_soff[j] = i_cur;
                    g_soff[j] = g_cur;
                }
                --left;
                --yl;
                if (yl != 0) {
                    i_cur += i_step;
                    g_cur += g_step;
                } else {
                    yl = ny;
                    --xl;
                    i_cur += i_rowjump;
                    g_cur += g_rowjump;
                    if (xl == 0) {
                        xl = nx;
                        i_cur += i_imgjump;
                        g_cur += g_imgjump;
                    }
                }
            }
        }
        // chunk q of the stage: part q % D1C of pixel q / D1C
#pragma unroll
        for (int q = 0; q < KCH; ++q) {
            const int slot_px = q >> d1c_shift, part = q - (slot_px << d1c_shift);
            int px = i_soff[0];
#pragma unroll
            for (int k = 1; k < KCH; ++k) px = slot_px == k ? i_soff[k] : px;
            copy_to_lds_dwords<CW>(rs_it, stage + (q * BM + 64 * wave) * 16, a_voff, px + part * CW * 4);
        }
#pragma unroll
        for (int j = 0; j < BPW; ++j) {
            const int q = wave * BPW + j;
            const int slot_px = q >> d1c_shift, part = q - (slot_px << d1c_shift);
            int px = g_soff[0];
#pragma unroll
            for (int k = 1; k < KCH; ++k) px = slot_px == k ? g_soff[k] : px;
            copy_to_lds_dwords<CW>(rs_gt, stage + A_BYTES + q * 1024, b_voff, px + part * CW * 4);
        }
    };

    float16v acc[TM];
    bool live[TM];  // row tiles of this wave that hold at least one real row
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        live[b] = it.row_tile * BM + 64 * wave + b * 32 < P.rows;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
    }
    float4v k4[KCH / 2], i4[KCH / 2][TM];

    static_for<NB - 1>([&](auto S0) { issue_stage(decltype(S0)::value); });
    __builtin_amdgcn_s_waitcnt(0x0F70 | KEEP);
    __syncthreads();
    for (int st = 0; st < nstages; st += NB) {  // surplus stages contract zeros
        static_for<NB>([&](auto SLOT) {
            constexpr int slot = decltype(SLOT)::value;
            const char* stage = smem + slot * STAGE_BYTES;
#pragma unroll
            for (int t = 0; t < KCH / 2; ++t) {  // lanes 0..31 take chunk 2t, lanes 32..63 chunk 2t+1
                k4[t] = *reinterpret_cast<const float4v*>(stage + A_BYTES + ((2 * t + h) * BN + lr) * 16);
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    i4[t][b] = *reinterpret_cast<const float4v*>(stage + ((2 * t + h) * BM + 64 * wave + b * 32 + lr) * 16);
            }
            issue_stage((slot + NB - 1) % NB);
#pragma unroll
            for (int t = 0; t < KCH / 2; ++t)
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    if (!live[b]) continue;  // wave-uniform
#pragma unroll
                    for (int u = 0; u < CW; ++u)
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[t][u], i4[t][b][u], acc[b], 0, 0, 0);
                }
            // this wave's copies of the next stage have landed, its reads of this stage are done;
            // after the barrier both hold for every wave
            __builtin_amdgcn_s_waitcnt((0x0F70 | KEEP) & 0xF0FF);
            __syncthreads();
        });
    }
    // the copies of the surplus stages still write (zeros) into this workgroup's LDS
    __builtin_amdgcn_s_waitcnt(0x0F70);

    float* __restrict__ out = P.out + (long long)it.split * P.out_elems;
    const long long caps = (long long)P.D0 * P.D2 * P.D3;
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const int R = it.row_tile * BM + 64 * wave + b * 32 + lr;
        if (R >= P.rows) continue;
        const int c = R / P.D2, d2 = R - c * P.D2;
        float* orow = out + ((long long)it.tap * P.C + c) * P.M * caps + ((long long)it.d0 * P.D2 + d2) * P.D3;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int j0 = 8 * g + 4 * h;  // registers 4g .. 4g+3 hold columns j0 .. j0+3
            if ((P.D3 & 3) == 0) {
                if (j0 < P.cols) {
                    const int m = j0 / P.D3, d3 = j0 - m * P.D3;
                    const float4v v = {acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]};
                    *reinterpret_cast<float4v*>(orow + (long long)m * caps + d3) = v;
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u, m = j / P.D3, d3 = j - m * P.D3;
                    if (j < P.cols) orow[(long long)m * caps + d3] = acc[b][4 * g + u];
                }
            }
        }
    }
}

struct Wgrad32Plan {
    Wgrad32Params P;
    int cw, tn, tm;
    int narrow_waves;  // wgrad32_narrow_kernel with that many waves; 0: wgrad32_kernel
    size_t it_bytes, gt_bytes, partial_bytes;
};

int ceil_div_i(long long a, long long b) { return (int)((a + b - 1) / b); }
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Valid floats per chunk: 4 or 3, such that a capsule column of D1 floats is 1, 2 or 4 chunks.
int chunk_width(const ConvShape& s)
{
    for (int cw : {4, 3}) {
        if (s.D1 % cw) continue;
        const int d1c = s.D1 / cw;
        if (d1c == 1 || d1c == 2 || d1c == 4) return cw;
    }
    return 0;
}

// Fewest ranges such that the images one range touches (N/nsplit + 3) stay below 0x7fffff00 bytes;
// 0 if a single image is already too large for that.
long long split_lower_bound(const ConvShape& s)
{
    const long long it_img = (long long)s.H * s.W * s.C * s.D0 * s.D1 * s.D2 * 4;
    const long long gt_img = (long long)s.Ho * s.Wo * s.M * s.D0 * s.D1 * s.D3 * 4;
    const long long img_max = it_img > gt_img ? it_img : gt_img;
    const long long imgs_cap = 0x7fffff00LL / (img_max > 0 ? img_max : 1);
    if (imgs_cap < 4) return 0;
    return (s.N + (imgs_cap - 3) - 1) / (imgs_cap - 3);
}

// Rows (columns) of `extent` that a tile of k MFMA tiles of 32 takes; 0: less than a capsule
int tile_step(int extent, int unit, int k)
{
    return extent > 32 * k ? 32 * k / unit * unit : 32 * k;  // several tiles: each begins at a whole capsule
}

// Tile: the least estimated time, of `steps` steps of 16 K values in every tile of all taps.  A wave splits
// TM + TN operands for TM x TN products: cost, in ns per 32 x 32 results and step with all SIMDs busy, is
// the mean of six capsule shapes with 576 rows and columns.  The code of a large tile takes time to arrive
// and to get under way: start, in us, is what tiny layers take more than with 1 x 1 tiles.  (By the fewest
// padded rows alone 150 x 220 took 1 x 1 tiles, 262 us at 12 GFLOP, now 161, and 96 x 384 with two dozen K
// values 3 x 3 ones, 22 us, now 13.)
double choose_tile(Wgrad32Params& P, double steps, int& tm, int& tn)
{
    static const double cost[3][3] = {{650, 470, 540}, {470, 360, 385}, {540, 385, 330}};
    static const double start[3][3] = {{0, 1.3, 4.5}, {1.5, 4, 8}, {5, 9, 15}};
    const int row_unit = P.natural ? P.D2 : 1, col_unit = P.natural ? P.D3 : 1;
    double best = -1;
    for (int a = 3; a >= 1; --a)
        for (int b = 3; b >= 1; --b) {
            const int rs = tile_step(P.rows, row_unit, a), cs = tile_step(P.cols, col_unit, b);
            if (rs == 0 || cs == 0) continue;
            const int rt = ceil_div_i(P.rows, rs), ct = ceil_div_i(P.cols, cs);
            const double busy = steps * P.ntaps * P.D0 * rt * ct * a * b * cost[a - 1][b - 1];
            const double time = start[a - 1][b - 1] + busy / (1024 * 1e3);  // 1024 SIMDs
            if (best >= 0 && time >= best) continue;
            best = time;
            tm = a; P.row_step = rs; P.row_tiles = rt;
            tn = b; P.col_step = cs; P.col_tiles = ct;
        }
    return best;
}

// Tiles and the split of the K loop (host side, pure arithmetic).
Wgrad32Plan make_plan(const ConvShape& s)
{
    Wgrad32Plan pl{};
    Wgrad32Params& P = pl.P;
    pl.cw = chunk_width(s);
    P.N = s.N; P.H = s.H; P.W = s.W; P.C = s.C; P.M = s.M; P.kw = s.kw; P.stride = s.stride;
    P.pad = s.pad; P.D0 = s.D0; P.D1 = s.D1; P.D2 = s.D2; P.D3 = s.D3; P.Ho = s.Ho; P.Wo = s.Wo;
    P.D1C = pl.cw ? s.D1 / pl.cw : 1;
    P.rows = s.C * s.D2;
    P.cols = s.M * s.D3;
    // square capsules need no transposed copies; their tiles begin at whole channels
    P.natural = s.D1 == s.D2 && s.D1 == s.D3;
    P.ntaps = s.kh * s.kw;
    const long long full = (long long)s.N * s.Ho * s.Wo;
    const double steps = (double)full * s.D1 / 16;  // of 16 K values, per tap
    if (!P.natural && P.cols <= 32) {
        pl.narrow_waves = P.rows <= 128 ? 2 : 4;
        P.row_step = 64 * pl.narrow_waves;
        P.row_tiles = ceil_div_i(P.rows, P.row_step);
        P.col_step = 32;
        P.col_tiles = 1;
    } else {
        choose_tile(P, steps, pl.tm, pl.tn);
    }
    P.tiles = P.ntaps * s.D0 * P.row_tiles * P.col_tiles;
    P.out_elems = (long long)s.kernel_elems();
    P.d3_magic = s.D3 > 1 && (long long)s.M * s.D3 * s.D3 < (1LL << 32)
                     ? (unsigned)(((1ULL << 32) + s.D3 - 1) / s.D3)
                     : 0u;  // 0: divide
    P.it_img_bytes = (long long)s.H * s.W * s.C * s.D0 * s.D1 * s.D2 * 4;
    P.gt_img_bytes = (long long)s.Ho * s.Wo * s.M * s.D0 * s.D1 * s.D3 * 4;
    pl.it_bytes = P.natural ? 0 : (size_t)s.N * P.it_img_bytes;
    pl.gt_bytes = P.natural ? 0 : (size_t)s.N * P.gt_img_bytes;

    // Split of the K loop (a tap's valid output pixels, at most N*Ho*Wo) over workgroups.  The
    // one-wave workgroups resident at a time are bounded by LDS and by registers (eight per CU where
    // 256 of them hold a tile, else four); the split aims at one full round of them and keeps at
    // least 8 stages per workgroup.  A range of N*rect/nsplit pixels touches at most N/nsplit + 3
    // images: their bytes must stay below 2^31 (a lower bound on nsplit), and the partial sums
    // below 1 GiB (an upper bound).
    long long per_cu, min_stages = 8;
    if (pl.narrow_waves) {
        const int kch = narrow_chunks(P.D1C, pl.narrow_waves);
        per_cu = 160 * 1024 / narrow_lds_bytes(pl.narrow_waves, kch);
        const int by_registers = (kch == 2 ? 12 : 8) / pl.narrow_waves;
        if (per_cu > by_registers) per_cu = by_registers;
        min_stages = kch == 2 ? 8 : 16;  // (of 4 chunks)
    } else {
        per_cu = 160 * 1024 / lds_bytes_of(pl.tm, pl.tn);
        const int by_registers = pl.tm + pl.tn <= 4 ? 8 : 4;
        if (per_cu > by_registers) per_cu = by_registers;
    }
    const long long slots = 256 * per_cu;
    long long want = slots / P.tiles;
    if (want < 1) want = 1;
    // more rounds where a range would be longer than 3072 K values (the rounding of a sum grows with
    // its length: 3x3x3 capsules, 32 channels, 64 images of 32x32: ranges of 5300 values 1.10e-6,
    // of 2660 7.8e-7; the fp32 instructions 1.05e-6)
    long long rounds = 1;
    while (rounds < 4 && full * s.D1 / (rounds * slots / P.tiles > 0 ? rounds * slots / P.tiles : 1) > 3072) ++rounds;
    if (rounds * slots / P.tiles > want) want = rounds * slots / P.tiles;
    // fewer where the reduction would take longer than the ranges gain: a wave takes about 1 us per 16 K
    // values, the reduction 0.04 us per range and 0.65 us per MB of partial sums (16x16 capsules, 3 -> 3
    // channels, 1x1 window, 440 thousand K values: 2048 ranges 138 us, 819 91)
    const double per_range = 0.04 + 0.65e-6 * 4.0 * (double)P.out_elems;
    long long enough = (long long)std::sqrt(steps / per_range);
    const long long precise = (full * s.D1 + 3071) / 3072;
    if (enough < precise) enough = precise;
    if (want > enough) want = enough;
    if (want < 1) want = 1;
    const long long min_pix = min_stages * SLOTS / P.D1C;
    if (want > (full + min_pix - 1) / min_pix) want = (full + min_pix - 1) / min_pix;
    if (want > 3072) want = 3072;
    while (want > 1 && (double)want * P.out_elems * 4 > (double)(1 << 30)) --want;
    const long long lo = split_lower_bound(s);
    if (want < lo) want = lo;
    P.nsplit = (int)want;
    P.items = (long long)P.nsplit * P.tiles;
    pl.partial_bytes = P.nsplit > 1 ? (size_t)P.nsplit * P.out_elems * sizeof(float) : 0;
    return pl;
}

template <int CW, int TM, int TN, int NAT>
hipError_t launch_one(const Wgrad32Params& P, hipStream_t stream)
{
    auto kern = wgrad32_kernel<CW, TM, TN, NAT>;
    constexpr int lds_bytes = lds_bytes_of(TM, TN);
    static std::atomic<unsigned long long> lds_set{0};
    hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), lds_bytes, lds_set);
    if (err != hipSuccess) return err;
    kern<<<dim3((unsigned)P.items), dim3(64), lds_bytes, stream>>>(P);
    return hipGetLastError();
}

template <int CW, int TM, int TN>
hipError_t launch_nat(const Wgrad32Params& P, hipStream_t stream)
{
    if (!P.natural) return launch_one<CW, TM, TN, 0>(P, stream);
    return P.D1C == 1 ? launch_one<CW, TM, TN, 1>(P, stream) : launch_one<CW, TM, TN, 2>(P, stream);
}

template <int CW, int NW, int KCH>
hipError_t launch_narrow(const Wgrad32Params& P, hipStream_t stream)
{
    auto kern = wgrad32_narrow_kernel<CW, NW, KCH>;
    constexpr int lds_bytes = narrow_lds_bytes(NW, KCH);
    static std::atomic<unsigned long long> lds_set{0};
    hipError_t err = set_dynamic_lds_once(reinterpret_cast<const void*>(kern), lds_bytes, lds_set);
    if (err != hipSuccess) return err;
    kern<<<dim3((unsigned)P.items), dim3(64 * NW), lds_bytes, stream>>>(P);
    return hipGetLastError();
}

template <int CW>
hipError_t launch_narrow(const Wgrad32Plan& pl, hipStream_t stream)
{
    if (pl.narrow_waves == 4) return launch_narrow<CW, 4, 4>(pl.P, stream);
    return pl.P.D1C == 4 ? launch_narrow<CW, 2, 4>(pl.P, stream) : launch_narrow<CW, 2, 2>(pl.P, stream);
}

template <int CW, int TM>
hipError_t launch_tn(const Wgrad32Plan& pl, hipStream_t stream)
{
    switch (pl.tn) {
        case 1: return launch_nat<CW, TM, 1>(pl.P, stream);
        case 2: return launch_nat<CW, TM, 2>(pl.P, stream);
        default: return launch_nat<CW, TM, 3>(pl.P, stream);
    }
}

template <int CW>
hipError_t launch_tm(const Wgrad32Plan& pl, hipStream_t stream)
{
    if (pl.narrow_waves) return launch_narrow<CW>(pl, stream);
    switch (pl.tm) {
        case 1: return launch_tn<CW, 1>(pl, stream);
        case 2: return launch_tn<CW, 2>(pl, stream);
        default: return launch_tn<CW, 3>(pl, stream);
    }
}

hipError_t launch_transpose32(const void* src, void* dst, size_t nmat, int A, int B,
                              hipStream_t stream)
{
    const size_t total = nmat * (size_t)A * B;
    const size_t blocks = (total + 1023) / 1024;
    if (blocks == 0 || blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    const float* from = static_cast<const float*>(src);
    float* to = static_cast<float*>(dst);
    if (total < 0xfffff000u)  // (the last threads' places too)
        transpose_caps32_kernel<unsigned><<<(unsigned)blocks, 256, 0, stream>>>(from, to, A, B, (unsigned)total);
    else
        transpose_caps32_kernel<size_t><<<(unsigned)blocks, 256, 0, stream>>>(from, to, A, B, total);
    return hipGetLastError();
}

}  // namespace

bool wgrad32_eligible(const ConvShape& s)
{
    if (s.dtype != 0) return false;
    if (chunk_width(s) == 0) return false;
    // 31-bit byte offsets within one image of either tensor, 31-bit counts
    const long long it_img = (long long)s.H * s.W * s.C * s.D0 * s.D1 * s.D2 * 4;
    const long long gt_img = (long long)s.Ho * s.Wo * s.M * s.D0 * s.D1 * s.D3 * 4;
    if (it_img >= (1LL << 31) || gt_img >= (1LL << 31)) return false;
    if ((long long)s.stride * s.W * s.C * s.D0 * s.D1 * s.D2 * 4 >= (1LL << 30)) return false;
    if ((long long)s.C * s.D2 >= (1 << 24) || (long long)s.M * s.D3 >= (1 << 24)) return false;
    const long long tiles = (long long)s.kh * s.kw * s.D0 * (((long long)s.C * s.D2 + 31) / 32) *
                            (((long long)s.M * s.D3 + 31) / 32);
    const long long lo = split_lower_bound(s);
    if (lo == 0 || lo > 3072) return false;
    if ((double)lo * (double)s.kernel_elems() * 4 > (double)(1 << 30) && lo > 1) return false;
    if (tiles * 3072 >= (1LL << 31)) return false;  // the split never exceeds 3072 ranges
    if ((long long)s.N * s.Ho * s.Wo >= (1LL << 31)) return false;  // pixel counts are 32-bit
    return true;
}

// A fit over 47 random layers of square capsules, 0.001 .. 38 GFLOP, 16 % root mean square: launches, the tiles'
// estimate (its scale is that of six layers of 576 rows and columns), and the partial sums of as many ranges as
// the reduction is worth.  The transposed copies of unequal capsules are not in it.
double wgrad32_us(const ConvShape& s)
{
    Wgrad32Params P{};
    int tm, tn;
    P.natural = s.D1 == s.D2 && s.D1 == s.D3;
    P.D2 = s.D2; P.D3 = s.D3; P.D0 = s.D0;
    P.rows = s.C * s.D2;
    P.cols = s.M * s.D3;
    P.ntaps = s.kh * s.kw;
    const double steps = (double)s.pixels() * s.D1 / 16;
    const double busy = choose_tile(P, steps, tm, tn);
    return 8.8 + 0.52 * busy + 0.99 * std::sqrt(steps * 4e-6 * (double)s.kernel_elems());
}

size_t wgrad32_workspace_bytes(const ConvShape& s)
{
    const Wgrad32Plan pl = make_plan(s);
    return align256(pl.it_bytes) + align256(pl.gt_bytes) + pl.partial_bytes;
}

hipError_t launch_wgrad32(const ConvShape& s, const void* input, const void* dout, float* dkernel,
                          void* workspace, hipStream_t stream)
{
    Wgrad32Plan pl = make_plan(s);
    char* ws = static_cast<char*>(workspace);
    void* it = ws;
    void* gt = ws + align256(pl.it_bytes);
    float* partial = reinterpret_cast<float*>(ws + align256(pl.it_bytes) + align256(pl.gt_bytes));
    hipError_t err = hipSuccess;
    if (pl.P.natural) {
        pl.P.it = input;
        pl.P.gt = dout;
    } else {
        err = launch_transpose32(input, it, (size_t)s.N * s.H * s.W * s.C * s.D0, s.D1, s.D2, stream);
        if (err != hipSuccess) return err;
        err = launch_transpose32(dout, gt, (size_t)s.N * s.Ho * s.Wo * s.M * s.D0, s.D1, s.D3, stream);
        if (err != hipSuccess) return err;
        pl.P.it = it;
        pl.P.gt = gt;
    }
    pl.P.out = pl.P.nsplit > 1 ? partial : dkernel;
    err = pl.cw == 3 ? launch_tm<3>(pl, stream) : launch_tm<4>(pl, stream);
    if (err != hipSuccess) return err;
    if (pl.P.nsplit > 1)
        err = launch_splitk_reduce(partial, dkernel, pl.P.out_elems, pl.P.nsplit, stream);
    return err;
}

}  // namespace capscaps
