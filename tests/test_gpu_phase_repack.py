"""Input gradients of strided 16-bit layers on the tuned kernels, whose phases' kernels are repacked in one launch where
the scratch holds them all, else one by one, against the CPU oracle: two to sixteen phases (empty ones among them), the
lane-per-row kernel and the large tiles, capsule rows that are read as 16-byte runs and others, and few columns, whose
padding leaves too little scratch for all phases together.  Integer operands: every partial sum is exact, so the
results equal the oracle's.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import capsconv
from paper_2104_02621_amd import workloads as wl
from tests.gpu_util import BWD_INPUT, NO_SMALL_TILES, repacks_together, route, run_op, to_device
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu
PHASES = 1  # the form's number in capscaps_testing_route

SHAPES = [
    ("s2", 3, 80, 80, 4, 8, 3, 3, 2, 1, 1, 8, 8, 8),
    ("s2_wide", 3, 80, 80, 33, 4, 3, 3, 2, 1, 1, 8, 8, 8),  # 264 columns of 512
    ("s2_one_row", 6, 80, 80, 4, 8, 1, 3, 2, 0, 1, 8, 8, 8),  # two phases, two without taps
    ("s2_d0", 6, 80, 78, 4, 5, 3, 3, 2, 1, 2, 8, 8, 8),
    ("s3", 12, 60, 61, 8, 8, 4, 3, 3, 1, 1, 8, 8, 8),
    ("s4", 24, 60, 59, 8, 8, 5, 4, 4, 1, 1, 8, 8, 8),
    ("s2_d4", 14, 80, 78, 4, 8, 3, 3, 2, 1, 1, 4, 4, 4),
    ("s2_d16", 4, 80, 62, 8, 6, 3, 3, 2, 1, 1, 16, 16, 16),
    ("s2_256", 3, 80, 80, 32, 2, 3, 3, 2, 1, 1, 8, 8, 8),
    ("s2_m1", 3, 80, 80, 32, 1, 3, 3, 2, 1, 1, 8, 8, 8),  # (16-bit results: a smaller kernel's scratch)
    ("s2_one_row_256", 6, 80, 80, 32, 2, 1, 3, 2, 0, 1, 8, 8, 8),
    ("s3_256", 12, 60, 61, 32, 2, 4, 3, 3, 1, 1, 8, 8, 8),
    ("s3_d4", 24, 60, 61, 60, 2, 4, 3, 3, 1, 1, 4, 4, 4),
    ("s4_256", 24, 60, 59, 32, 2, 5, 4, 4, 1, 1, 8, 8, 8),
    ("s4_d16", 12, 60, 59, 16, 1, 5, 4, 4, 1, 1, 16, 16, 16),
]
# results in 32 bits, in 16: which of them one launch repacks
TOGETHER = ({"s2_wide", "s2_d0", "s2_d4", "s2_d16", "s2_256", "s2_m1", "s2_one_row_256", "s3_256", "s3_d4", "s4_256", "s4_d16"},
            {"s2_wide", "s2_d0", "s2_d16", "s2_256", "s2_one_row_256", "s3_256", "s4_256", "s4_d16"})


def test_the_shapes_take_the_phases():
    for s in SHAPES:
        w = small(s[0], wl.BF16, *s[1:])
        for out16, together in enumerate(TOGETHER):
            assert route(w, BWD_INPUT, NO_SMALL_TILES, out16)[2] == PHASES, s[0]
            assert repacks_together(w, NO_SMALL_TILES, out16) == (s[0] in together), (s[0], out16)


@pytest.mark.parametrize("out16", [False, True], ids=["out32", "out16"])
@pytest.mark.parametrize("dtype", [wl.BF16, wl.FP16], ids=["bf16", "fp16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
def test_input_gradient_equals_the_oracle(shape, dtype, out16):
    import torch
    w = wl.integer_variant(small(shape[0], dtype, *shape[1:], seed=len(shape[0]) + 80))
    _, k_st, _, k32 = wl.generate(w)
    g_st, g32 = wl.generate_dout(w)
    ref = torch.from_numpy(capsconv.conv_bwd_input(g32, k32, (w.H, w.W), w.stride, w.pad))
    k_dev, g_dev = to_device(k_st, w.dtype), to_device(g_st, w.dtype)
    got = run_op(w, BWD_INPUT, g_dev, k_dev, NO_SMALL_TILES, out16=out16).cpu()
    assert ref.abs().max() < 2 ** 24
    expected = ref.float().to(got.dtype)
    assert np.array_equal(got.float().numpy(), expected.float().numpy()), w.name
