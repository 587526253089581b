"""GPU parity of the fp32 kernel that contracts on the bf16 matrix instructions (every operand as
the sum of three bf16 values): tile edges of every column-tile count and both chunk widths, whole and
split K loops, and the values the decomposition cannot hold, which a workgroup recomputes on the
fp32 instructions.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl
from tests.gpu_util import run_gpu, shape_args, to_device
from tests.test_gpu_parity import full_compare, small

pytestmark = pytest.mark.gpu

# (N, H, W, C, M, kh, kw, stride, pad, D0, D1, D2, D3): column tiles of 1 .. 4 with the last one
# ragged, capsule columns of 3 (stored by runs of three registers), 6 and 9 and not, K loops that
# end inside a period of stages, 256-row and 64-row tiles
SHAPES = [
    (3, 7, 9, 5, 3, 3, 3, 1, 1, 3, 3, 3, 3),     # 9 columns: one tile of 10 capsules
    (3, 7, 9, 5, 11, 3, 3, 1, 1, 1, 3, 3, 3),    # 33: two tiles' worth in 20 capsules
    (2, 9, 8, 4, 27, 2, 3, 2, 1, 2, 2, 3, 3),    # 81: three, ragged
    (2, 6, 7, 7, 43, 3, 1, 1, 0, 1, 3, 6, 3),    # 129: past 42 capsules of four tiles
    (2, 8, 8, 3, 7, 3, 3, 1, 1, 1, 5, 12, 6),    # D3 = 6
    (2, 8, 8, 3, 5, 3, 3, 1, 1, 1, 2, 4, 9),     # D3 = 9
    (2, 8, 8, 3, 7, 3, 3, 1, 1, 1, 3, 3, 12),    # D3 = 12: a multiple of 4 as well
    (4, 9, 9, 6, 9, 3, 3, 1, 1, 1, 4, 4, 4),     # 36
    (2, 9, 9, 3, 25, 3, 3, 2, 2, 1, 8, 8, 4),    # 100: four tiles, two kernel stages in the ring
    (2, 9, 9, 5, 17, 1, 1, 1, 0, 1, 4, 16, 5),   # 85, stored element by element
    (1, 5, 5, 1, 1, 3, 3, 1, 0, 1, 1, 4, 4),     # a single row tile, nearly empty
    (20, 24, 24, 3, 6, 3, 3, 1, 1, 1, 4, 3, 5),  # more than 560 tiles of 64 rows: one-wave tiles
    (70, 33, 32, 2, 4, 3, 3, 1, 1, 1, 1, 4, 4),  # more than 256 tiles of 256 rows
    (20, 24, 24, 3, 8, 3, 3, 1, 1, 1, 4, 4, 4),  # one-wave tiles of one column tile, 4-float chunks ...
    (24, 24, 24, 2, 10, 3, 3, 1, 1, 1, 3, 3, 3),  # ... and stored by runs of three
]


@pytest.mark.parametrize("integers", [False, True], ids=["normal", "integers"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_split_kernel_matches_oracle(shape, integers):
    w = small("split_" + "x".join(map(str, shape)), wl.FP32, *shape, seed=611)
    full_compare(wl.integer_variant(w) if integers else w, cc.PATH_MFMA_TUNED32)


def exact64(w, x, k):
    from oracle import capsconv
    with np.errstate(invalid="ignore", over="ignore"):
        return capsconv.conv_fwd(x, k, w.stride, w.pad)


SPECIAL = [(2, 9, 9, 4, 9, 3, 3, 1, 1, 1, 4, 4, 4), (2, 9, 9, 5, 9, 3, 3, 1, 1, 3, 3, 3, 3)]


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, -3.4028235e38, 3.3961775e38])
@pytest.mark.parametrize("shape", SPECIAL, ids=["4x4", "3x3x3"])
@pytest.mark.parametrize("side", ["input", "kernel"])
def test_values_bf16_cannot_hold(shape, value, side):
    """One infinity, NaN or value that rounds to infinity in bf16: the results it does not reach are
    untouched, those it reaches are what fp32 arithmetic gives."""
    if side == "kernel":  # no padding: a matrix core multiplies a padding tap's zeros by the kernel
        shape = shape[:8] + (0,) + shape[9:]
    w = small("special", wl.FP32, *shape, seed=612)
    x, k, _, _ = wl.generate(w)
    x, k = x.copy(), k.copy()
    k *= np.float32(0.125)  # a product with the largest fp32 value stays finite
    x = np.clip(x, -1, 1)
    (x if side == "input" else k).flat[37] = value
    ref = exact64(w, x, k)
    got = run_gpu(w, to_device(x, wl.FP32), to_device(k, wl.FP32), cc.PATH_MFMA_TUNED32).cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf].astype(np.float32))
    ok = np.isfinite(ref) & (np.abs(ref) < 3e38)
    assert ok.any() and np.isfinite(got[ok]).all()
    # fp32 sums of K <= 180 terms, relative to the largest result of the capsule's magnitude
    scale = np.maximum(np.abs(ref[ok]), np.abs(ref[np.isfinite(ref) & (np.abs(ref) < 1e3)]).max())
    assert (np.abs(got[ok] - ref[ok]) / scale).max() <= 180 * 2.0 ** -24


@pytest.mark.parametrize("shape", SPECIAL, ids=["4x4", "3x3x3"])
@pytest.mark.parametrize("scale", [1e-36, 3e-38, 1e-30, 1e30])
def test_results_of_any_magnitude(shape, scale):
    """The same relative error at every magnitude of the input (1e-36: the third bf16 term of most
    values is below bf16's range)."""
    w = small("magnitude", wl.FP32, *shape, seed=613)
    x, k, _, _ = wl.generate(w)
    x = (x.astype(np.float64) * scale).astype(np.float32)
    ref = exact64(w, x, k)
    got = run_gpu(w, to_device(x, wl.FP32), to_device(k, wl.FP32), cc.PATH_MFMA_TUNED32).cpu().numpy()
    # products below 2^-126 are rounded to multiples of 2^-149
    floor = 180 * 2.0 ** -149
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max() + floor


# ---- kernel gradient on the same decomposition: tiles of 1 .. 3 by 1 .. 3 MFMA tiles (several of
# them beginning at whole capsules), both chunk widths, one, two and four chunks per capsule column,
# square capsules (read in place) and others (transposed copies), ranges long enough to change sign
WGRAD_SHAPES = [
    (3, 7, 9, 5, 3, 3, 3, 1, 1, 3, 3, 3, 3),       # 15 x 9
    (2, 8, 7, 22, 33, 2, 2, 1, 0, 1, 3, 3, 3),     # 66 x 99: several tiles of whole 3-row capsules
    (2, 6, 6, 11, 17, 3, 3, 2, 1, 1, 6, 6, 6),     # 66 x 102, two 3-float chunks
    (1, 5, 6, 3, 9, 2, 2, 1, 1, 1, 12, 12, 12),    # 36 x 108, four 3-float chunks
    (2, 9, 9, 7, 25, 3, 3, 1, 1, 1, 4, 4, 4),      # 28 x 100
    (2, 7, 7, 13, 9, 3, 3, 1, 2, 1, 8, 8, 8),      # 104 x 72
    (2, 6, 5, 5, 4, 2, 2, 1, 0, 2, 16, 16, 16),    # 80 x 64, four 4-float chunks
    (3, 9, 7, 20, 14, 3, 3, 1, 1, 1, 6, 5, 4),     # 100 x 56, transposed
    (2, 9, 7, 9, 13, 3, 3, 3, 1, 1, 4, 5, 7),      # 45 x 91, transposed, stride 3
    (40, 20, 20, 4, 5, 1, 1, 1, 0, 1, 4, 4, 4),    # ranges of many stages
]

# transposed copies and at most 32 columns: two and four waves per workgroup on the fp32 instructions, one,
# two and four chunks of 3 and 4 floats per capsule column, 32 columns and fewer, stored by fours and one by one
WGRAD_SHAPES += [
    (3, 9, 7, 20, 8, 3, 3, 1, 1, 1, 6, 5, 4),       # 100 x 32
    (2, 8, 9, 43, 5, 3, 3, 2, 1, 2, 3, 4, 6),       # 172 x 30, four waves
    (2, 7, 7, 3, 2, 3, 2, 1, 1, 1, 12, 5, 7),       # 15 x 14, four chunks, two waves
    (5, 6, 5, 70, 4, 2, 2, 1, 0, 1, 4, 4, 8),       # 280 x 32, two row tiles
    (2, 6, 5, 9, 2, 3, 3, 1, 1, 1, 16, 16, 3),      # 144 x 6, four chunks, four waves
    (2, 9, 9, 33, 1, 1, 1, 3, 0, 1, 8, 2, 1),       # 66 x 1
    (40, 16, 16, 4, 3, 1, 1, 1, 0, 1, 4, 5, 4),     # ranges of many stages
]


def wgrad(w, x, g):
    return cc.conv_bwd_kernel(to_device(x, wl.FP32), to_device(g, wl.FP32), (w.kh, w.kw), w.stride,
                              w.pad).cpu().numpy()


@pytest.mark.parametrize("shape", WGRAD_SHAPES, ids=["x".join(map(str, s)) for s in WGRAD_SHAPES])
def test_split_kernel_gradient_matches_oracle(shape):
    from oracle import capsconv
    w = small("splitw_" + "x".join(map(str, shape)), wl.FP32, *shape, seed=614)
    for v in (w, wl.integer_variant(w)):
        x = wl.generate(v)[0]
        g = wl.generate_dout(v)[0]
        ref = capsconv.conv_bwd_kernel(x, g, (v.kh, v.kw), v.stride, v.pad)
        got = wgrad(v, x, g)
        if v is w:
            # random sums of n terms: 2^-24 sqrt(n) of their size, n <= 16000
            assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
        else:
            assert np.array_equal(got, ref)


@pytest.mark.parametrize("value", [np.inf, np.nan, -3.4028235e38])
@pytest.mark.parametrize("shape", [(2, 9, 9, 4, 9, 3, 3, 1, 0, 1, 4, 4, 4), (2, 9, 9, 5, 9, 3, 3, 1, 0, 3, 3, 3, 3)],
                         ids=["4x4", "3x3x3"])
def test_kernel_gradient_of_values_bf16_cannot_hold(shape, value):
    from oracle import capsconv
    w = small("specialw", wl.FP32, *shape, seed=615)
    x = np.clip(wl.generate(w)[0], -1, 1)
    g = np.clip(wl.generate_dout(w)[0], -1, 1) * np.float32(0.125)
    x.flat[53] = value
    with np.errstate(invalid="ignore", over="ignore"):
        ref = capsconv.conv_bwd_kernel(x, g, (w.kh, w.kw), w.stride, w.pad)
    got = wgrad(w, x, g)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf].astype(np.float32))
    ok = np.isfinite(ref) & (np.abs(ref) < 1e30)
    assert ok.any() and np.abs(got[ok] - ref[ok]).max() <= 1e-5 * np.abs(ref[ok]).max()
    big = np.isfinite(ref) & (np.abs(ref) >= 1e30) & (np.abs(ref) < 3e38)
    assert (np.abs(got[big] - ref[big]) <= 1e-5 * np.abs(ref[big])).all()


# ---- fp32 capsule rows no 12- or 16-byte copy fits: layers large enough to be written out in runs
# of four K values first (D2 = 1, 2, 5, 7, 9), one part and several, forward and through the
# transposed kernel view of the input gradient
RECHUNK_SHAPES = [
    (12, 20, 17, 11, 14, 5, 5, 1, 2, 1, 6, 5, 4),
    (40, 24, 24, 9, 17, 3, 3, 2, 1, 2, 4, 7, 3),
    (40, 24, 24, 18, 34, 3, 3, 2, 1, 2, 4, 7, 3),
    (60, 28, 28, 33, 12, 3, 3, 1, 0, 1, 2, 1, 5),
    (30, 32, 32, 13, 18, 3, 3, 1, 1, 1, 5, 2, 9),
]


@pytest.mark.parametrize("shape", RECHUNK_SHAPES, ids=["x".join(map(str, s)) for s in RECHUNK_SHAPES])
def test_rows_of_any_length_match_oracle(shape):
    w = small("rechunk_" + "x".join(map(str, shape)), wl.FP32, *shape, seed=616)
    assert w.flops_nominal() >= 1.2e9
    full_compare(w, cc.PATH_AUTO)


def test_input_written_out_in_several_parts():
    """150 MB of input: parts of 48 MiB, the last one shorter; small integers, so every kernel gives
    the same bits."""
    w = wl.integer_variant(small("parts", wl.FP32, 230, 40, 41, 10, 6, 3, 3, 1, 1, 1, 2, 5, 4, seed=617))
    x, k = (to_device(t, wl.FP32) for t in wl.generate(w)[:2])
    assert np.prod(w.input_shape) * 4 > 2 * (48 << 20)
    a = run_gpu(w, x, k, cc.PATH_AUTO)
    b = run_gpu(w, x, k, cc.PATH_DIRECT)
    assert bool((a == b).all())


@pytest.mark.parametrize("shape", [(24, 16, 18, 12, 10, 3, 3, 1, 1, 1, 6, 4, 5), (30, 15, 15, 8, 12, 5, 5, 2, 2, 1, 4, 8, 7)])
def test_input_gradient_with_rows_of_any_length(shape):
    from oracle import capsconv
    w = small("rechunk_dx", wl.FP32, *shape, seed=618)
    k = wl.generate(w)[1]
    g = wl.generate_dout(w)[0]
    ref = capsconv.conv_bwd_input(g, k, (w.H, w.W), w.stride, w.pad)
    got = cc.conv_bwd_input(to_device(g, wl.FP32), to_device(k, wl.FP32), (w.H, w.W), w.stride, w.pad)
    assert np.abs(got.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()


# ---- operands of opposite magnitudes: what a split drops of a tiny operand is multiplied by the other
# one, so a result of ordinary size may rest on it, and a kernel tensor may be as small as an input
MAGNITUDES = [(1, 1e-36), (1, 1e-39), (1, 1e-41), (1e-36, 1e30), (1e30, 1e-36), (1e-38, 1e20), (1e20, 1e-38),
              (1e-40, 1e35), (1e35, 1e-40), (1e-41, 1), (1e15, 1e15), (1e-44, 1e30)]


def scaled(a, scale):
    return (a.astype(np.float64) * scale).astype(np.float32)


def check_magnitude(got, ref):
    # sums of fp32 products: 1e-5 of the largest result, and below 2^-126 multiples of 2^-149 (one
    # rounding per addition at most, fewer than 4000 of them)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max() + 4000 * 2.0 ** -149


@pytest.mark.parametrize("scales", MAGNITUDES, ids=lambda s: f"{s[0]:g}x{s[1]:g}")
@pytest.mark.parametrize("shape", SPECIAL + [(12, 20, 17, 11, 14, 5, 5, 1, 2, 1, 6, 5, 4)],
                         ids=["4x4", "3x3x3", "rows_of_5"])
def test_forward_with_operands_of_any_magnitude(shape, scales):
    w = small("magnitudes", wl.FP32, *shape, seed=619)
    x, k = (scaled(a, s) for a, s in zip(wl.generate(w)[:2], scales))
    path = cc.PATH_AUTO if shape[12] == 4 and shape[11] == 5 else cc.PATH_MFMA_TUNED32
    got = run_gpu(w, to_device(x, wl.FP32), to_device(k, wl.FP32), path).cpu().numpy()
    check_magnitude(got, exact64(w, x, k))


@pytest.mark.parametrize("scales", MAGNITUDES, ids=lambda s: f"{s[0]:g}x{s[1]:g}")
def test_input_gradient_with_operands_of_any_magnitude(scales):
    from oracle import capsconv
    w = small("magnitudes_dx", wl.FP32, 24, 18, 18, 16, 16, 3, 3, 1, 1, 1, 3, 3, 3, seed=620)
    args = (w.N, w.H, w.W, w.M, w.C, w.kh, w.kw, 1, 1, w.D0, w.D1, w.D3, w.D2, w.dtype)
    assert cc.capscaps_select_path(*args) == cc.PATH_MFMA_TUNED32
    k = scaled(wl.generate(w)[1], scales[1])
    g = scaled(wl.generate_dout(w)[0], scales[0])
    got = cc.conv_bwd_input(to_device(g, wl.FP32), to_device(k, wl.FP32), (w.H, w.W), w.stride, w.pad)
    check_magnitude(got.cpu().numpy(), capsconv.conv_bwd_input(g, k, (w.H, w.W), w.stride, w.pad))


@pytest.mark.parametrize("scales", MAGNITUDES, ids=lambda s: f"{s[0]:g}x{s[1]:g}")
@pytest.mark.parametrize("shape", [WGRAD_SHAPES[0], WGRAD_SHAPES[4], WGRAD_SHAPES[7]],
                         ids=["3x3x3", "4x4", "6x5.5x4"])
def test_kernel_gradient_with_operands_of_any_magnitude(shape, scales):
    from oracle import capsconv
    w = small("magnitudes_dk", wl.FP32, *shape, seed=621)
    x = scaled(wl.generate(w)[0], scales[0])
    g = scaled(wl.generate_dout(w)[0], scales[1])
    check_magnitude(wgrad(w, x, g), capsconv.conv_bwd_kernel(x, g, (w.kh, w.kw), w.stride, w.pad))


# ---- long K loops, unsplit: the bf16 instructions drop bits toward minus infinity
@pytest.mark.parametrize("shape", [(16, 23, 23, 128, 2, 8, 8, 1, 0, 1, 16, 16, 4), (128, 19, 19, 43, 3, 8, 8, 1, 0, 1, 4, 12, 3)],
                         ids=["K131072", "K33024"])
def test_errors_of_long_sums_have_no_direction(shape):
    import torch
    N, H, W, C, M, kh, kw, _, _, _, D1, D2, D3 = shape
    K, Ho, Wo = kh * kw * C * D2, H - kh + 1, W - kw + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(622)
    x = torch.randn((N, H, W, C, 1, D1, D2), generator=gen, device="cuda")
    k = torch.randn((kh, kw, C, M, 1, D2, D3), generator=gen, device="cuda") / K ** 0.5
    ref = torch.zeros((N * Ho * Wo * D1, M * D3), dtype=torch.float64, device="cuda")
    for p in range(kh):
        for q in range(kw):
            rows = x[:, p:p + Ho, q:q + Wo, :, 0].permute(0, 1, 2, 4, 3, 5).reshape(-1, C * D2)
            ref += rows.double() @ k[p, q, :, :, 0].permute(0, 2, 1, 3).reshape(C * D2, M * D3).double()
    got = cc.conv_fwd(x, k, 1, 0, path=cc.PATH_MFMA_TUNED32)
    err = got[:, :, :, :, 0].permute(0, 1, 2, 4, 3, 5).reshape(-1, M * D3).double() - ref
    rms, mean = err.pow(2).mean().sqrt().item(), err.mean().item()
    print(f"K {K}: rms error {rms:.2e}, mean {mean:+.2e}", flush=True)
    # Sums of N(0,1) size, one rounding (at most 2^-24 of the partial sum, evenly distributed: 0.58 of it)
    # per accumulation of a bf16 instruction, 6 per 16 K values; partial sums grow as sqrt(k / K).
    n = 6 * K / 16
    assert rms <= 0.58 * 2 ** -24 * (n / 2) ** 0.5 * 1.5
    # what is dropped, 2^-9 of the last bit (2^-23) per instruction on average, cancels but for the last
    # 96 stages of 16 (12) K values at most: 576 instructions; the mean of independent errors, over
    # 500000 results, is far below that
    assert abs(mean) <= 576 * 2 ** -9 * 2 ** -23 + 5 * rms / err.numel() ** 0.5


def test_forced_any_shape_kernel_runs_on_rows_of_any_length():
    """The any-shape kernel, forced, gives an image the same bits in a batch of 20 and in one of 640: it
    adds up the K values in one order.  The library's own choice for the large batch, which contracts
    bf16 terms, does not."""
    import torch
    big = small("generic_rows", wl.FP32, 640, 32, 32, 2, 8, 3, 3, 1, 1, 2, 1, 5, 5, seed=623)
    few = small("generic_rows", wl.FP32, 20, 32, 32, 2, 8, 3, 3, 1, 1, 2, 1, 5, 5, seed=623)
    assert big.flops_nominal() >= 1.2e9
    assert cc.capscaps_select_path(*shape_args(big)) == cc.PATH_MFMA
    x, k = (to_device(t, wl.FP32) for t in wl.generate(big)[:2])
    ref = run_gpu(few, x[:20].contiguous(), k, cc.PATH_MFMA_GENERIC)
    assert torch.equal(run_gpu(big, x, k, cc.PATH_MFMA_GENERIC)[:20], ref)
    own = run_gpu(big, x, k, cc.PATH_MFMA)
    assert torch.equal(run_gpu(big, x, k, cc.PATH_AUTO), own) and not torch.equal(own[:20], ref)
