"""The passes that lay fp32 operands out anew before they are contracted on bf16 instructions, against the CPU oracle: the
kernel packed by pairs of values (pairs that span two channels, an odd number of K values), and the transposed
capsules written four at a time (counts that leave one to three).  Integer operands: sums are exact, but an integer is
its first bf16 term alone; so the packed kernel also with real values.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import capsconv
from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl
from tests.gpu_util import BWD_KERNEL, FWD, NO_SMALL_TILES, route, run_op, to_device
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

PACKED = [  # 1.2 GFLOP and more: rows are written out in runs of four K values first; 12- and 16-byte rows as they are
    ("d1", 6, 24, 23, 37, 16, 3, 3, 1, 1, 1, 8, 1, 12),
    ("d5", 4, 20, 21, 11, 16, 3, 3, 1, 1, 2, 6, 5, 6),
    ("d7", 4, 20, 21, 9, 14, 3, 3, 1, 1, 1, 9, 7, 8),
    ("d3", 12, 24, 25, 13, 17, 3, 2, 1, 1, 3, 3, 3, 3),
    ("d4", 12, 24, 25, 13, 17, 3, 3, 1, 1, 1, 4, 4, 5),
]
TRANSPOSED = [
    ("one_over", 1, 5, 5, 3, 3, 3, 3, 1, 1, 1, 3, 5, 5),
    ("three_over", 3, 5, 7, 1, 1, 2, 2, 1, 0, 1, 3, 1, 7),
    ("two_over", 1, 3, 7, 1, 3, 1, 1, 1, 0, 1, 6, 5, 3),
    ("d12", 2, 7, 6, 3, 5, 3, 3, 2, 1, 2, 12, 4, 3),
]


@pytest.mark.parametrize("shape", PACKED, ids=[s[0] for s in PACKED])
def test_packed_kernel(shape):
    w = wl.integer_variant(small(shape[0], wl.FP32, *shape[1:], seed=90))
    i_st, k_st, i32, k32 = wl.generate(w)
    ref = capsconv.conv_fwd(i32, k32, w.stride, w.pad)
    got = run_op(w, FWD, to_device(i_st, w.dtype), to_device(k_st, w.dtype), NO_SMALL_TILES)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), ref)


def rms(a):
    return float(np.sqrt(np.mean(np.square(a, dtype=np.float64))))


@pytest.mark.parametrize("shape", PACKED, ids=[s[0] for s in PACKED])
def test_packed_kernel_of_real_values(shape):
    """All three terms of every value count: without its third one the kernel tensor would be off by up to 2^-17 of
    each value, the results by several times the bound."""
    w = small(shape[0], wl.FP32, *shape[1:], seed=92)
    i_st, k_st, i32, k32 = wl.generate(w)
    ref = capsconv.conv_fwd(i32, k32, w.stride, w.pad)
    got = run_op(w, FWD, to_device(i_st, w.dtype), to_device(k_st, w.dtype), NO_SMALL_TILES).cpu().numpy()
    # one rounding (0.58 of 2^-24 of a partial sum, which grow as sqrt(k / K)) per accumulation, 6 per 16 K values
    bound = 0.58 * 2.0 ** -24 * (3 * w.kh * w.kw * w.C * w.D2 / 16) ** 0.5 * 1.5 * rms(ref)
    assert rms(got - ref) <= bound

    def bf16(a):  # to nearest even
        u = a.astype(np.float32).view(np.uint32)
        return ((u + 0x7fff + (u >> 16 & 1)) & 0xffff0000).view(np.float32)
    first = bf16(k32)
    two_terms = first + bf16(k32 - first)
    assert rms(capsconv.conv_fwd(i32, two_terms, w.stride, w.pad) - ref) > 3 * bound


def test_the_layers_take_the_packed_kernel_and_the_transposed_copies():
    for s in PACKED:
        packed = cc.PATH_MFMA_TUNED32 if s[0] in ("d3", "d4") else cc.PATH_MFMA  # (rows written out: reported as the latter)
        assert route(small(s[0], wl.FP32, *s[1:]), FWD, NO_SMALL_TILES)[::2] == (-1, packed), s[0]
    for s in TRANSPOSED:
        assert s[11:] != (s[11],) * 3  # square capsules are read in place
        assert route(small(s[0], wl.FP32, *s[1:]), BWD_KERNEL, NO_SMALL_TILES)[::2] == (-1, 32), s[0]


@pytest.mark.parametrize("shape", TRANSPOSED, ids=[s[0] for s in TRANSPOSED])
def test_transposed_capsules(shape):
    w = wl.integer_variant(small(shape[0], wl.FP32, *shape[1:], seed=91))
    i_st, _, i32, _ = wl.generate(w)
    g_st, g32 = wl.generate_dout(w)
    ref = capsconv.conv_bwd_kernel(i32, g32, (w.kh, w.kw), w.stride, w.pad)
    got = run_op(w, BWD_KERNEL, to_device(i_st, w.dtype), to_device(g_st, w.dtype), NO_SMALL_TILES)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), ref)
