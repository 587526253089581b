"""The small-tile kernels (16-bit forward pass, input gradient in one launch, kernel gradient) at the
sizes where they can go wrong: tiles of one row and one column and their remainders, K loops shorter than the
ring of stages, odd channel counts with 4-element rows, every capsule shape's copy layout, leading
capsule indices, strided phases (with and without pixels no window reaches), non-square windows, splits of
the K loop; small-integer data, so that every result is exact, and infinities at the image border."""
import numpy as np
import pytest

from oracle import capsconv
from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl

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
          (1, 20, 20, 64, 2, 3, 3, 1, 1, (1, 8, 8, 8)), (300, 3, 3, 2, 2, 3, 3, 1, 1, (1, 4, 4, 4))]


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
    got = cc.conv_bwd_kernel(_gpu(i32, dtype), _gpu(g32, dtype), (3, 3), 1, 1)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    inside = np.zeros((3, 3), bool)
    inside[1:, 1:] = True
    assert np.isposinf(got[inside]).all()
    assert np.isfinite(got[~inside]).all()


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
