"""Helpers shared by the GPU parity tests: upload seeded inputs, call the C ABI through the
binding, bring results back, and the error measures the tolerances are stated in."""
import ctypes

import numpy as np

from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl

# Tolerances.  The target is max|g-r| / max|r| <= 1e-5 for fp32 and <= 2e-2 for 16-bit inputs
# with fp32 accumulation.  16-bit products are exact in fp32, so for every dtype the only
# error source is the order of fp32 additions; against the scale S = sum|I*K| of each output
# that error is bounded by about (number of terms) * 2^-24 in the worst case and is of order
# sqrt(terms) * 2^-24 for random data, so a second, much sharper check err/S <= 1e-5 is made
# for all dtypes (terms <= 9216 in every test here: worst-case bound 5.5e-4, typical 6e-6).
TOL_PRIMARY = {wl.FP32: 1e-5, wl.BF16: 2e-2, wl.FP16: 2e-2}
TOL_VS_ABS_SUM = 1e-5


def to_device(storage: np.ndarray, dtype: int):
    import torch
    if dtype == wl.BF16:
        return torch.from_numpy(storage.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(storage).cuda()


def shape_args(w: wl.Workload):
    return (w.N, w.H, w.W, w.C, w.M, w.kh, w.kw, w.stride, w.pad, w.D0, w.D1, w.D2, w.D3, w.dtype)


def run_gpu(w: wl.Workload, i_dev, k_dev, path=cc.PATH_AUTO, out=None, workspace=None):
    """One call through capscaps_conv_fwd_path on torch's current stream -> device tensor."""
    import torch
    if out is None:
        # poison the output so that an element the kernel fails to write cannot pass
        out = torch.full(w.out_shape, float("nan"), dtype=torch.float32, device="cuda")
    need = cc.capscaps_conv_fwd_workspace_bytes(*shape_args(w))
    if workspace is None:
        workspace = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    rc = cc.capscaps_conv_fwd_path(i_dev.data_ptr(), k_dev.data_ptr(), out.data_ptr(), w.N, w.H,
                                   w.W, w.C, w.M, w.kh, w.kw, w.stride, w.pad, w.D0, w.D1, w.D2,
                                   w.D3, w.dtype, path, workspace.data_ptr(), workspace.numel(),
                                   torch.cuda.current_stream().cuda_stream)
    assert rc == cc.OK, f"{w.name}: status {rc} ({cc.capscaps_strerror(rc)}; {cc.capscaps_last_hip_error()})"
    return out


def errors(got: np.ndarray, ref: np.ndarray, abs_sum: np.ndarray):
    """(max|g-r| / max|r|,  max(|g-r| / S))."""
    assert got.shape == ref.shape, (got.shape, ref.shape)
    assert np.isfinite(got).all(), "non-finite values (or unwritten outputs) in the GPU result"
    diff = np.abs(got.astype(np.float64) - ref)
    primary = diff.max() / max(np.abs(ref).max(), 1e-300)
    secondary = (diff / np.maximum(abs_sum, 1e-300)).max()
    return float(primary), float(secondary)


def check(w: wl.Workload, got, ref, abs_sum, label=""):
    primary, secondary = errors(got, ref, abs_sum)
    msg = f"{w.name} {label}: rel-to-max {primary:.3e}, rel-to-abs-sum {secondary:.3e}"
    print(msg, flush=True)
    assert primary <= TOL_PRIMARY[w.dtype], msg
    assert secondary <= TOL_VS_ABS_SUM, msg
    return primary, secondary


# The small-tile kernels of a call: by the library's rules, none, or wherever they can run with a given tile
# (an index) and pieces of the K loop.  Test entry points of the library, not in its header.
BY_RULE, NO_SMALL_TILES = (0, -1, 0), (1, -1, 0)
FWD, BWD_INPUT, BWD_KERNEL = 0, 1, 2


def small_tiles(tile=-1, pieces=0):
    return (2, tile, pieces)


def _ints(values):
    return (ctypes.c_int * len(values))(*values)


def route(w: wl.Workload, op, tiles=BY_RULE, out16=False, workspace_bytes=1 << 40):
    """(tile of the small-tile kernel or -1, its pieces of the K loop, path / form of the other kernels)."""
    info = _ints([0, 0, 0])
    fn = cc._load().capscaps_testing_route
    fn.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    rc = fn(op, _ints(shape_args(w)), int(out16), _ints(tiles), workspace_bytes, info)
    assert rc == cc.OK, rc
    return tuple(info)


def repacks_together(w: wl.Workload, tiles=BY_RULE, out16=False):
    """Does one launch repack the kernels of this input gradient's phases?"""
    fn = cc._load().capscaps_testing_repacks_together
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    return bool(fn(_ints(shape_args(w)), int(out16), _ints(tiles)))


def run_op(w: wl.Workload, op, a_dev, b_dev, tiles=BY_RULE, out16=False):
    """A forward pass or gradient with the given use of the small-tile kernels -> device tensor."""
    import torch
    args = shape_args(w)
    shape = (w.out_shape, w.input_shape, w.kernel_shape)[op]
    need = ((cc.capscaps_conv_fwd_out16_workspace_bytes if out16 else cc.capscaps_conv_fwd_workspace_bytes),
            (cc.capscaps_conv_bwd_input_out16_workspace_bytes if out16 else cc.capscaps_conv_bwd_input_workspace_bytes),
            cc.capscaps_conv_bwd_kernel_workspace_bytes)[op](*args)
    out = torch.full(shape, float("nan"), dtype=a_dev.dtype if out16 else torch.float32, device="cuda")
    # (partial sums of the pieces a test asks for, behind what the size query covers)
    ws = torch.empty(need + 16 + 4 * max(tiles[2], 0) * out.numel(), dtype=torch.uint8, device="cuda")
    fn = cc._load().capscaps_testing_conv
    p, i = ctypes.c_void_p, ctypes.c_int
    fn.argtypes = [i, p, i, p, p, p, p, p, ctypes.c_size_t, p]
    rc = fn(op, _ints(args), int(out16), _ints(tiles), a_dev.data_ptr(), b_dev.data_ptr(), out.data_ptr(),
            ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == cc.OK, f"{w.name}: status {rc} ({cc.capscaps_strerror(rc)}; {cc.capscaps_last_hip_error()})"
    return out
