"""The small-tile kernels (16-bit forward pass, input gradient in one launch, kernel gradient) at the
sizes where they can go wrong: tiles of one row and one column and their remainders, K loops shorter than the
ring of stages, odd channel counts with 4-element rows, every capsule shape's copy layout, leading
capsule indices, strided phases (with and without pixels no window reaches), non-square windows; every layer with
the library's own choice and with every tile, with and without a split K loop; small-integer data, so that every
result is exact, and infinities at the image border."""
import numpy as np
import pytest

from oracle import capsconv
from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl
from tests.gpu_util import BWD_INPUT, BWD_KERNEL, FWD, route, run_op, small_tiles

pytestmark = pytest.mark.gpu

#        N   H   W   C   M  kh kw  s  p  caps
SHAPES = [(1, 1, 1, 1, 1, 1, 1, 1, 0, (1, 4, 4, 4)), (1, 3, 3, 1, 2, 3, 3, 1, 1, (1, 4, 4, 4)),
          (2, 7, 5, 3, 5, 3, 3, 1, 1, (1, 4, 4, 4)), (3, 9, 8, 7, 17, 5, 5, 1, 2, (1, 4, 4, 4)),
          (2, 9, 9, 6, 4, 3, 3, 2, 1, (1, 4, 4, 4)), (2, 6, 6, 33, 3, 6, 6, 1, 0, (1, 4, 4, 4)),
          (1, 5, 5, 2, 1, 3, 3, 1, 0, (1, 8, 8, 8)), (2, 8, 7, 3, 9, 3, 3, 1, 1, (1, 8, 8, 8)),
          (3, 9, 10, 5, 8, 4, 4, 2, 1, (1, 8, 8, 8)), (1, 11, 6, 40, 17, 3, 3, 1, 1, (1, 8, 8, 8)),
          (2, 9, 9, 3, 5, 1, 1, 2, 0, (1, 8, 8, 8)), (2, 8, 9, 3, 4, 2, 3, 1, 1, (1, 8, 8, 8)),
          (1, 6, 6, 2, 3, 3, 3, 1, 1, (1, 16, 16, 16)), (2, 10, 10, 5, 1, 3, 3, 3, 2, (1, 16, 16, 16)),
          (5, 4, 4, 4, 6, 4, 4, 1, 0, (1, 16, 16, 16)), (2, 9, 7, 3, 5, 3, 3, 1, 1, (1, 1, 8, 16)),
          (9, 6, 6, 7, 2, 5, 5, 1, 2, (1, 1, 8, 16)), (2, 11, 11, 4, 3, 3, 3, 2, 1, (1, 1, 8, 16)),
          (3, 7, 7, 5, 3, 3, 3, 1, 1, (1, 4, 8, 16)), (2, 12, 5, 3, 2, 6, 6, 2, 3, (1, 4, 8, 16)),
          (2, 6, 5, 3, 2, 3, 3, 1, 1, (2, 8, 8, 8)), (2, 5, 5, 3, 4, 3, 3, 2, 1, (3, 4, 4, 4)),
          (2, 5, 6, 3, 2, 3, 3, 1, 1, (1, 2, 8, 32)), (4, 6, 6, 3, 2, 5, 5, 1, 4, (1, 2, 16, 8)),
          (1, 20, 20, 64, 2, 3, 3, 1, 1, (1, 8, 8, 8)), (300, 3, 3, 2, 2, 3, 3, 1, 1, (1, 4, 4, 4)),
          # more than 128 rows and columns in every operation, with remainders; without padding a kernel
          # gradient's 128-row tiles hold rows of two window taps
          (2, 7, 6, 35, 37, 3, 2, 1, 0, (1, 4, 4, 4)), (2, 7, 6, 18, 19, 2, 2, 1, 0, (1, 8, 8, 8)),
          (1, 6, 5, 9, 10, 3, 3, 1, 0, (1, 16, 16, 16)), (40, 3, 3, 21, 9, 2, 2, 1, 0, (1, 1, 8, 16)),
          (21, 4, 3, 9, 19, 3, 3, 1, 1, (1, 2, 16, 8)), (9, 5, 4, 19, 9, 2, 3, 2, 1, (1, 4, 8, 16))]
# tiles of the forward pass and input gradient, and of the kernel gradient (igemm_mid.hip, wgrad_mid.hip)
TILES = {FWD: 5, BWD_INPUT: 5, BWD_KERNEL: 4}


def _id(s):
    return "x".join(map(str, s[:9])) + "_" + ".".join(map(str, s[9]))


def _layer(shape, dtype):
    N, H, W, C, M, kh, kw, s, p, caps = shape
    return wl.Workload("mid_tiles", dtype, N, H, W, C, M, kh, kw, s, p, *caps, "int", "int", 0.0, 1201, 1202)


def _data(w):
    rng = np.random.default_rng(77)
    draw = lambda shape: rng.integers(-2, 3, size=shape).astype(np.float32)
    return draw(w.input_shape), draw(w.kernel_shape), draw(w.out_shape)


def _gpu(a, dtype):
    import torch
    return torch.from_numpy(a).cuda().to({wl.FP32: torch.float32, wl.BF16: torch.bfloat16, wl.FP16: torch.float16}[dtype])


@pytest.mark.parametrize("dtype", [wl.FP32, wl.BF16, wl.FP16], ids=["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", SHAPES, ids=_id)
def test_small_tiles_on_integers(shape, dtype):
    import torch
    w = _layer(shape, dtype)
    i32, k32, g32 = _data(w)
    I, K, G = (_gpu(a, dtype) for a in (i32, k32, g32))
    refs = {"out": capsconv.conv_fwd(i32, k32, w.stride, w.pad),
            "dx": capsconv.conv_bwd_input(g32, k32, (w.H, w.W), w.stride, w.pad),
            "dk": capsconv.conv_bwd_kernel(i32, g32, (w.kh, w.kw), w.stride, w.pad)}
    for out16 in (False,) if dtype == wl.FP32 else (False, True):
        got = {"out": cc.conv_fwd(I, K, w.stride, w.pad, out16=out16),
               "dx": cc.conv_bwd_input(G, K, (w.H, w.W), w.stride, w.pad, out16=out16),
               "dk": cc.conv_bwd_kernel(I, G, (w.kh, w.kw), w.stride, w.pad)}
        torch.cuda.synchronize()
        for name, t in got.items():
            # sums of integers are exact in fp32 (|sum| < 2^24); the 16-bit results are those, rounded once
            want = torch.from_numpy(refs[name].astype(np.float32)).to(t.dtype)
            assert torch.equal(t.cpu(), want.reshape(t.shape)), (w.name, name, out16)


def _can_run(w, op):
    """Capsules that the small-tile kernels take."""
    D1, D2, D3 = w.D1, w.D2, w.D3
    taps = 1 if (w.kh, w.kw, w.pad) == (w.H, w.W, 0) else w.kh * w.kw  # (fully connected: one 1x1 convolution)
    if op == BWD_INPUT and taps * w.M * D3 <= 24:
        return False  # (so short a sum takes the wavefront-level path, on a kernel tensor laid out for it)
    if w.dtype == wl.FP32:
        return op != FWD and D2 >= 4 and D3 >= 4
    return (D1, D2, D3) == (4, 4, 4) or D2 >= 8 and D3 >= 8


@pytest.mark.parametrize("dtype", [wl.FP32, wl.BF16, wl.FP16], ids=["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", SHAPES, ids=_id)
def test_every_tile_and_split_on_integers(shape, dtype):
    import torch
    w = _layer(shape, dtype)
    i32, k32, g32 = _data(w)
    I, K, G = (_gpu(a, dtype) for a in (i32, k32, g32))
    refs = {FWD: capsconv.conv_fwd(i32, k32, w.stride, w.pad),
            BWD_INPUT: capsconv.conv_bwd_input(g32, k32, (w.H, w.W), w.stride, w.pad),
            BWD_KERNEL: capsconv.conv_bwd_kernel(i32, g32, (w.kh, w.kw), w.stride, w.pad)}
    operands = {FWD: (I, K), BWD_INPUT: (G, K), BWD_KERNEL: (I, G)}
    for op in (FWD, BWD_INPUT, BWD_KERNEL):
        ref = torch.from_numpy(refs[op].astype(np.float32))
        for tile in range(TILES[op]):
            for pieces in (1, 3):
                for out16 in (False, True) if dtype != wl.FP32 and op != BWD_KERNEL else (False,):
                    ask = small_tiles(tile, pieces)
                    runs = route(w, op, ask, out16)
                    assert runs[0] in ((tile,) if _can_run(w, op) else (-1,)), (w.name, op, runs)
                    got = run_op(w, op, *operands[op], ask, out16)
                    torch.cuda.synchronize()
                    assert torch.equal(got.cpu(), ref.to(got.dtype).reshape(got.shape)), (w.name, op, ask, out16)


@pytest.mark.parametrize("dtype", [wl.FP32, wl.BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("caps", [(1, 4, 4, 4), (1, 8, 8, 8), (1, 1, 8, 16)], ids=str)
def test_infinities_stay_with_the_taps_that_meet_them(caps, dtype):
    """An infinite output gradient at a corner pixel reaches only the kernel gradient's taps that lie inside the
    image there: it never meets the zeros of the padding."""
    import torch
    w = _layer((2, 6, 6, 3, 4, 3, 3, 1, 1, caps), dtype)
    i32, k32, g32 = _data(w)
    i32 = np.abs(i32) + 1
    g32[0, 0, 0] = np.inf
    I, G = _gpu(i32, dtype), _gpu(g32, dtype)
    inside = np.zeros((3, 3), bool)
    inside[1:, 1:] = True
    got = [cc.conv_bwd_kernel(I, G, (3, 3), 1, 1)]
    for tile in range(TILES[BWD_KERNEL]):  # (tiles of 128 rows: a tap's rows rounded up to whole tiles)
        assert route(w, BWD_KERNEL, small_tiles(tile))[0] == tile
        got.append(run_op(w, BWD_KERNEL, I, G, small_tiles(tile)))
    torch.cuda.synchronize()
    for dk in got:
        dk = dk.cpu().numpy()
        assert np.isposinf(dk[inside]).all()
        assert np.isfinite(dk[~inside]).all()


#                                N  H   W  C  M  kh kw s  p  caps
@pytest.mark.parametrize("shape", [(2, 6, 5, 3, 4, 1, 3, 1, 1, (1, 8, 8, 8)), (2, 5, 5, 3, 4, 3, 3, 1, 4, (1, 4, 4, 4)),
                                   (1, 9, 8, 5, 12, 3, 2, 1, 1, (2, 4, 8, 8)), (2, 9, 7, 3, 4, 3, 4, 2, 2, (1, 4, 4, 4)),
                                   (20, 24, 23, 18, 16, 1, 5, 1, 2, (1, 8, 8, 8))], ids=_id)
@pytest.mark.parametrize("dtype", [wl.FP32, wl.BF16, wl.FP16], ids=["fp32", "bf16", "fp16"])
def test_infinite_weights_reach_only_their_pixels(shape, dtype):
    """Input gradients of non-square windows and of paddings beyond k - 1 are sums over the taps inside the image: an
    infinite and a NaN kernel value reach the pixels that these taps reach and no others."""
    import torch
    w = _layer(shape, dtype)
    rng = np.random.default_rng(78)
    k32 = rng.integers(1, 4, size=w.kernel_shape).astype(np.float32)
    g32 = rng.integers(1, 3, size=w.out_shape).astype(np.float32)
    k32[0, 0, 0, 0, 0, 0, 0] = np.inf
    k32[-1, -1, 1, 1, 0, 1, 1] = np.nan
    finite = np.where(np.isfinite(k32), k32, 0).astype(np.float32)
    want = capsconv.conv_bwd_input(g32, finite, (w.H, w.W), w.stride, w.pad)
    reach = lambda bad: capsconv.conv_bwd_input(g32, bad.astype(np.float32), (w.H, w.W), w.stride, w.pad) > 0
    want[reach(np.isinf(k32))] = np.inf
    want[reach(np.isnan(k32))] = np.nan
    assert np.isfinite(want).any() and np.isinf(want).any() and np.isnan(want).any()
    for out16 in (False,) if dtype == wl.FP32 else (False, True):
        got = cc.conv_bwd_input(_gpu(g32, dtype), _gpu(k32, dtype), (w.H, w.W), w.stride, w.pad, out16=out16)
        torch.cuda.synchronize()
        ref = torch.from_numpy(want.astype(np.float32)).to(got.dtype).reshape(got.shape)
        assert torch.equal(got.cpu().nan_to_num(nan=-1.0, posinf=-2.0), ref.nan_to_num(nan=-1.0, posinf=-2.0)), out16


@pytest.mark.parametrize("dtype", [wl.BF16, wl.FP16], ids=["bf16", "fp16"])
@pytest.mark.parametrize("N,C,M,D,pieces", [(30, 8, 8, 4, 200), (3, 64, 34, 8, 1)], ids=["200_pieces", "one_long_chain"])
def test_long_sums_have_short_chains_of_roundings(N, C, M, D, pieces, dtype):
    """A sum of n terms of random sign, one rounding (2.5e-8 of the value, root mean square) per term, is off by
    2.5e-8 sqrt(n / 2): 1.4e-7 for chains of 64 partial sums, and with as much again for chains of 32 matrix
    instructions, whose roundings are not all to nearest, below 2e-7.  As one chain, 200 partial sums or the instructions of
    486 stages are off by 2.5e-7 and 3.9e-7."""
    import torch
    H = 36
    w = wl.Workload("chains", dtype, N, H, H, C, M, 1, 1, 1, 0, 1, D, D, D, "normal", "normal", 1.0, 5, 6)
    gen = torch.Generator().manual_seed(9)
    I, G = (torch.randn(s, generator=gen).to({wl.BF16: torch.bfloat16, wl.FP16: torch.float16}[dtype]).cuda()
            for s in (w.input_shape, w.out_shape))
    got = run_op(w, BWD_KERNEL, I, G, small_tiles(0, pieces)).double().cpu()
    rows = lambda t, ch: t.double().cpu().view(-1, ch, D, D).permute(0, 2, 1, 3).reshape(-1, ch * D)
    ref = (rows(I, C).t() @ rows(G, M)).view(C, D, M, D).permute(0, 2, 1, 3).reshape(got.shape)
    error = float((got - ref).norm() / ref.norm())
    print(f"{pieces} pieces: {error:.3e}", flush=True)
    assert error < 2e-7
