"""Performance cases of the capsule convolution: what a program that uses this library has it do.

A case is one layer (forward, backward, or a training step of both) or the five-layer stack of
`workloads.net5` (inference or a training step), always through the library's public entry points:
single layers through the C names with the output and the workspace the program keeps, as
`bench.py` and a C caller do; the stack through the tensor functions `conv_fwd`, `conv_bwd_input`
and `conv_bwd_kernel`, which allocate their results.

`listed()` holds fixed cases; `draw(rng)` makes more of the ranges they stand for.
"""
import math
from types import SimpleNamespace

import torch

from paper_2104_02621_amd import capscaps as cc
from paper_2104_02621_amd import workloads as wl

TORCH_DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}
CODE = {"fp32": cc.FP32, "bf16": cc.BF16, "fp16": cc.FP16}


def _layer(name, op, dtype, N, H, W, C, M, k, stride, pad, caps, out16=False):
    D0, D1, D2, D3 = caps
    kh, kw = (k, k) if isinstance(k, int) else k
    return {"name": name, "kind": "layer", "op": op, "dtype": dtype, "out16": out16, "N": N, "H": H,
            "W": W, "C": C, "M": M, "kh": kh, "kw": kw, "stride": stride, "pad": pad, "D0": D0,
            "D1": D1, "D2": D2, "D3": D3}


def listed():
    return [
        # The smallest layer in use (benchmark configuration 1): a few microseconds of work, where
        # launches and latency are everything.
        _layer("fwd_fp32_small", "fwd", "fp32", 8, 16, 16, 4, 4, 3, 1, 0, (1, 4, 4, 4)),
        # The class-capsule layer at the end of a network (benchmark configuration 4): the window
        # covers the whole image.  Inference, then a training step of the same layer.
        _layer("fwd_fp32_fc", "fwd", "fp32", 256, 6, 6, 32, 10, 6, 1, 0, (1, 4, 4, 4)),
        _layer("train_fp32_fc", "train", "fp32", 256, 6, 6, 32, 10, 6, 1, 0, (1, 4, 4, 4)),
        # 3x3x3 capsules as in the paper's worked example (benchmark configuration 2), both ways.
        _layer("fwd_fp32_3d", "fwd", "fp32", 64, 32, 32, 32, 32, 3, 1, 1, (3, 3, 3, 3)),
        _layer("bwd_fp32_3d", "bwd", "fp32", 64, 32, 32, 32, 32, 3, 1, 1, (3, 3, 3, 3)),
        # An odd fp32 layer: 31x27 images, capsules of unequal extents, channel counts that fill no
        # tile, a 5x5 window; a training step.
        _layer("train_fp32_ragged", "train", "fp32", 20, 31, 27, 20, 14, 5, 1, 2, (1, 6, 5, 4)),
        # A strided 16-bit layer of 8x8 capsules (benchmark configuration 3), both ways; the
        # gradient handed to the layer below is in the storage type, as in a stack.
        _layer("fwd_bf16_strided", "fwd", "bf16", 128, 28, 28, 64, 64, 3, 2, 1, (1, 8, 8, 8)),
        _layer("bwd_bf16_strided", "bwd", "bf16", 128, 28, 28, 64, 64, 3, 2, 1, (1, 8, 8, 8), True),
        # Matrix capsules: 4x4 poses, 32 channels on 14x14 images, the middle of a small network;
        # a training step.
        _layer("train_bf16_4x4", "train", "bf16", 32, 14, 14, 32, 32, 3, 1, 1, (1, 4, 4, 4), True),
        # The largest layer (benchmark configuration 5).
        _layer("fwd_fp16_large", "fwd", "fp16", 64, 32, 32, 64, 64, 3, 1, 1, (1, 16, 16, 16)),
        # The five-layer stack: one image through it, as a server answers a request, and a
        # training step over a batch (forward, then every gradient training needs).
        {"name": "stack_infer_one", "kind": "stack", "op": "infer", "dtype": "bf16", "N": 1},
        {"name": "stack_train", "kind": "stack", "op": "train", "dtype": "bf16", "N": 64},
    ]


def draw(rng):
    """One more case of the ranges above: batch 1 .. 256, images 4 .. 40, 2 .. 96 channels, windows
    1 .. 6 and the whole image, strides 1 and 2, the capsule shapes the tests and the benchmark
    use, every direction and element type."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if rng.random() < 0.12:
        return {"kind": "stack", "op": rng.choice(["infer", "train"]),
                "dtype": rng.choice(["bf16", "fp16"]), "N": log_int(1, 64)}
    while True:
        dtype = rng.choice(["fp32", "bf16", "fp16"])
        if dtype == "fp32":
            caps = rng.choice([(3, 3, 3, 3), (1, 4, 4, 4), (1, 4, 4, 4), (1, 8, 8, 8), (1, 6, 5, 4),
                               (1, 1, 8, 16), (2, 4, 4, 4)])
        else:
            caps = rng.choice([(1, 4, 4, 4), (1, 8, 8, 8), (1, 8, 8, 8), (1, 16, 16, 16),
                               (1, 4, 8, 16), (1, 1, 8, 16)])
        C, M = log_int(2, 96), log_int(2, 96)
        if rng.random() < 0.6:  # most programs use multiples of 8
            C, M = max(8, C // 8 * 8), max(8, M // 8 * 8)
        H = rng.randint(4, 40)
        W = H if rng.random() < 0.7 else rng.randint(4, 40)
        N = log_int(1, 256)
        if rng.random() < 0.15:  # a fully-connected layer
            H = W = rng.randint(1, 8)
            k, stride, pad = H, 1, 0
        else:
            k = rng.choice([1, 3, 3, 3, 5, 6])
            stride = rng.choice([1, 1, 2])
            pad = rng.choice([0, k // 2])
        if k > min(H, W) + 2 * pad:
            continue
        op = rng.choice(["fwd", "fwd", "bwd", "train"])
        out16 = dtype != "fp32" and rng.random() < 0.5
        case = _layer("", op, dtype, N, H, W, C, M, k, stride, pad, caps, out16)
        del case["name"]
        w = work(case)
        if 1e6 <= w["flops"] <= (2e11 if dtype == "fp32" else 2e12) and w["bytes"] <= 2e9:
            return case


# --------------------------------------------------------------------------------------- shapes
def _geometry(case):
    g = SimpleNamespace(**{k: v for k, v in case.items() if k not in ("name", "kind", "op")})
    g.Ho = (g.H + 2 * g.pad - g.kh) // g.stride + 1
    g.Wo = (g.W + 2 * g.pad - g.kw) // g.stride + 1
    g.args = (g.N, g.H, g.W, g.C, g.M, g.kh, g.kw, g.stride, g.pad, g.D0, g.D1, g.D2, g.D3,
              CODE[g.dtype])
    g.in_shape = (g.N, g.H, g.W, g.C, g.D0, g.D1, g.D2)
    g.k_shape = (g.kh, g.kw, g.C, g.M, g.D0, g.D2, g.D3)
    g.out_shape = (g.N, g.Ho, g.Wo, g.M, g.D0, g.D1, g.D3)
    return g


def _stack_layers(case):
    """The stack's layers as cases (forward output 16-bit but for the last layer's)."""
    return [_layer("", "", case["dtype"], w.N, w.H, w.W, w.C, w.M, (w.kh, w.kw), w.stride, w.pad,
                   (w.D0, w.D1, w.D2, w.D3), i < 4)
            for i, w in enumerate(wl.net5(case["N"], CODE[case["dtype"]]))]


def _randn(gen, shape, sigma, dtype):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    return x.mul_(sigma).to(TORCH_DTYPE[dtype])


def _layer_inputs(case, seed):
    """Input N(0,1), kernel N(0, 1/fan-in), output gradient N(0,1), in the layer's element type."""
    g = _geometry(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = _randn(gen, g.in_shape, 1.0, g.dtype)
    k = _randn(gen, g.k_shape, 1.0 / math.sqrt(g.kh * g.kw * g.C * g.D2), g.dtype)
    dout = _randn(gen, g.out_shape, 1.0, g.dtype) if case["op"] != "fwd" else None
    return g, x, k, dout


def _stack_inputs(case, seed):
    layers = [_geometry(c) for c in _stack_layers(case)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = _randn(gen, layers[0].in_shape, 1.0, case["dtype"])
    kernels = [_randn(gen, g.k_shape, 1.0 / math.sqrt(g.kh * g.kw * g.C * g.D2), g.dtype)
               for g in layers]
    dout = _randn(gen, layers[-1].out_shape, 1.0, case["dtype"]) if case["op"] == "train" else None
    return layers, x, kernels, dout


# ------------------------------------------------------------------------------- prepare and run
def prepare(case, seed):
    if case["kind"] == "stack":
        layers, x, kernels, dout = _stack_inputs(case, seed)
        return SimpleNamespace(kind="stack", op=case["op"], layers=layers, x=x, kernels=kernels,
                               dout=dout)
    g, x, k, dout = _layer_inputs(case, seed)
    small = TORCH_DTYPE[g.dtype] if g.out16 else torch.float32
    st = SimpleNamespace(kind="layer", op=case["op"], g=g, x=x, k=k, dout=dout)
    need = 16
    if st.op != "bwd":
        st.out = torch.empty(g.out_shape, dtype=small, device="cuda")
        need = max(need, (cc.capscaps_conv_fwd_out16_workspace_bytes if g.out16 else
                          cc.capscaps_conv_fwd_workspace_bytes)(*g.args))
    if st.op != "fwd":
        st.dx = torch.empty(g.in_shape, dtype=small, device="cuda")
        st.dk = torch.empty(g.k_shape, dtype=torch.float32, device="cuda")
        need = max(need, (cc.capscaps_conv_bwd_input_out16_workspace_bytes if g.out16 else
                          cc.capscaps_conv_bwd_input_workspace_bytes)(*g.args))
        need = max(need, cc.capscaps_conv_bwd_kernel_workspace_bytes(*g.args))
    # the calls of one pass run one after the other on one stream and share the workspace
    st.ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    return st


def _ok(status):
    if status != cc.OK:
        raise cc.CapscapsError(status)


def run(st):
    if st.kind == "stack":
        return _run_stack(st)
    g, ws, n = st.g, st.ws.data_ptr(), st.ws.numel()
    stream = torch.cuda.current_stream().cuda_stream
    outputs = {}
    if st.op != "bwd":
        fwd = cc.capscaps_conv_fwd_out16 if g.out16 else cc.capscaps_conv_fwd_ex
        _ok(fwd(st.x.data_ptr(), st.k.data_ptr(), st.out.data_ptr(), *g.args, ws, n, stream))
        outputs["out"] = st.out
    if st.op != "fwd":
        bwd = cc.capscaps_conv_bwd_input_out16 if g.out16 else cc.capscaps_conv_bwd_input
        _ok(bwd(st.dout.data_ptr(), st.k.data_ptr(), st.dx.data_ptr(), *g.args, ws, n, stream))
        _ok(cc.capscaps_conv_bwd_kernel(st.x.data_ptr(), st.dout.data_ptr(), st.dk.data_ptr(),
                                        *g.args, ws, n, stream))
        outputs["dx"] = st.dx
        outputs["dk"] = st.dk
    return outputs


def _run_stack(st):
    acts = [st.x]
    for g, k in zip(st.layers, st.kernels):
        acts.append(cc.conv_fwd(acts[-1], k, g.stride, g.pad, out16=g.out16))
    outputs = {"out": acts[-1]}
    if st.op == "train":
        grad = st.dout
        for i in range(len(st.layers) - 1, -1, -1):
            g = st.layers[i]
            outputs[f"dk{i + 1}"] = cc.conv_bwd_kernel(acts[i], grad, (g.kh, g.kw), g.stride, g.pad)
            if i > 0:  # the first layer's input needs no gradient
                grad = cc.conv_bwd_input(grad, st.kernels[i], (g.H, g.W), g.stride, g.pad,
                                         out16=True)
    return outputs


# -------------------------------------------------------------------------------------- the work
def _taps_inside(extent, out_extent, k, stride, pad):
    return sum(0 <= o * stride - pad + t < extent for o in range(out_extent) for t in range(k))


def work(case):
    """Multiply-adds against real input pixels only (padding is no work); every operand read once
    and every result written once."""
    if case["kind"] == "stack":
        layers = [_geometry(c) for c in _stack_layers(case)]
        flops = total = 0
        for i, g in enumerate(layers):
            f, b = _layer_sizes(g)
            train = case["op"] == "train"
            flops += f * (1 + (2 if i > 0 else 1) if train else 1)
            total += b["k"] + (4 * b["nk"] if train else 0)
        total += _layer_sizes(layers[0])[1]["in"]
        out = _layer_sizes(layers[-1])[1]
        return {"bytes": total + 4 * out["nout"] + (out["dout"] if case["op"] == "train" else 0),
                "flops": flops}
    g = _geometry(case)
    f, b = _layer_sizes(g)
    res = b["es"] if g.out16 else 4
    fwd, bwd = case["op"] != "bwd", case["op"] != "fwd"
    total = b["in"] + b["k"]
    total += res * b["nout"] if fwd else 0
    total += b["dout"] + res * b["nin"] + 4 * b["nk"] if bwd else 0
    return {"bytes": total, "flops": f * (fwd + 2 * bwd)}


def _layer_sizes(g):
    taps = (_taps_inside(g.H, g.Ho, g.kh, g.stride, g.pad) *
            _taps_inside(g.W, g.Wo, g.kw, g.stride, g.pad))
    flops = 2 * g.N * taps * g.M * g.D0 * g.D1 * g.D3 * g.C * g.D2
    es = 4 if g.dtype == "fp32" else 2
    nin, nk, nout = math.prod(g.in_shape), math.prod(g.k_shape), math.prod(g.out_shape)
    return flops, {"es": es, "nin": nin, "nk": nk, "nout": nout, "in": es * nin, "k": es * nk,
                   "dout": es * nout}


def tolerance(case):
    """About four times what the library's results measure against `exact` over the listed and 26
    drawn cases: fp32 results 1e-7 .. 2.2e-6 (single values up to 1.4e-5 of the result's size),
    results rounded once to the storage type 1.7e-3 (bf16) and 2.1e-4 (fp16).  In the stack the
    activations handed on are rounded, and a sum taken in another order rounds some of them the
    other way: 1.3e-3 in bf16, single values 1.1e-2."""
    if case["kind"] == "stack":
        return {"rel": 5e-3, "max": 4.5e-2} if case["dtype"] == "bf16" else {"rel": 7e-4, "max": 6e-3}
    if case["out16"]:
        return {"rel": 7e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 9e-4, "max": 2e-3}
    return {"rel": 1e-5, "max": 6e-5}


# ------------------------------------------------------------------------------ 64-bit reference
def _rows(t, d0):
    """[N,x,y,ch,D0,D1,Dk] -> the matrix [(N,x,y,D1), (ch,Dk)] of leading index d0."""
    s = t[:, :, :, :, d0].permute(0, 1, 2, 4, 3, 5).contiguous()
    return s.view(-1, s.shape[4] * s.shape[5])


def _from_rows(mat, n, x, y, ch, d1, dk):
    return mat.view(n, x, y, d1, ch, dk).permute(0, 1, 2, 4, 3, 5)


def _padded(x, g):
    xp = torch.zeros((g.N, g.H + 2 * g.pad, g.W + 2 * g.pad) + tuple(x.shape[3:]),
                     dtype=torch.float64, device=x.device)
    xp[:, g.pad:g.pad + g.H, g.pad:g.pad + g.W] = x
    return xp


def _window(xp, g, p, q):
    return xp[:, p:p + g.stride * (g.Ho - 1) + 1:g.stride, q:q + g.stride * (g.Wo - 1) + 1:g.stride]


def _kernel_matrix(k, g, p, q, d0):
    """[(C,D2), (M,D3)]"""
    return k[p, q, :, :, d0].permute(0, 2, 1, 3).double().reshape(g.C * g.D2, g.M * g.D3)


def _taps(g):
    return [(p, q, d0) for p in range(g.kh) for q in range(g.kw) for d0 in range(g.D0)]


def _exact_fwd(g, x, k):
    xp = _padded(x, g)
    acc = [0.0] * g.D0
    for p, q, d0 in _taps(g):
        acc[d0] = acc[d0] + _rows(_window(xp, g, p, q), d0) @ _kernel_matrix(k, g, p, q, d0)
    out = torch.empty(g.out_shape, dtype=torch.float64, device=x.device)
    for d0 in range(g.D0):
        out[:, :, :, :, d0] = _from_rows(acc[d0], g.N, g.Ho, g.Wo, g.M, g.D1, g.D3)
    return out


def _exact_bwd_input(g, dout, k):
    dxp = torch.zeros((g.N, g.H + 2 * g.pad, g.W + 2 * g.pad, g.C, g.D0, g.D1, g.D2),
                      dtype=torch.float64, device=dout.device)
    grad = [_rows(dout, d0).double() for d0 in range(g.D0)]
    for p, q, d0 in _taps(g):
        da = grad[d0] @ _kernel_matrix(k, g, p, q, d0).t().contiguous()
        _window(dxp, g, p, q)[:, :, :, :, d0] += _from_rows(da, g.N, g.Ho, g.Wo, g.C, g.D1, g.D2)
    return dxp[:, g.pad:g.pad + g.H, g.pad:g.pad + g.W].contiguous()


def _exact_bwd_kernel(g, x, dout):
    xp = _padded(x, g)
    dk = torch.empty(g.k_shape, dtype=torch.float64, device=x.device)
    grad = [_rows(dout, d0).double() for d0 in range(g.D0)]
    for p, q, d0 in _taps(g):
        db = _rows(_window(xp, g, p, q), d0).t() @ grad[d0]
        dk[p, q, :, :, d0] = db.view(g.C, g.D2, g.M, g.D3).permute(0, 2, 1, 3)
    return dk


def exact(case, seed):
    """The same sums in 64 bits; between the layers of the stack the activations and gradients are
    rounded to the storage type, as the 16-bit-output entry points do."""
    if case["kind"] == "stack":
        layers, x, kernels, dout = _stack_inputs(case, seed)
        acts = [x]
        for g, k in zip(layers, kernels):
            y = _exact_fwd(g, acts[-1], k)
            acts.append(y.to(x.dtype) if g.out16 else y)
        outputs = {"out": acts[-1]}
        if case["op"] == "train":
            grad = dout
            for i in range(len(layers) - 1, -1, -1):
                outputs[f"dk{i + 1}"] = _exact_bwd_kernel(layers[i], acts[i], grad)
                if i > 0:
                    grad = _exact_bwd_input(layers[i], grad, kernels[i]).to(x.dtype)
        return outputs
    g, x, k, dout = _layer_inputs(case, seed)
    outputs = {}
    if case["op"] != "bwd":
        outputs["out"] = _exact_fwd(g, x, k)
    if case["op"] != "fwd":
        outputs["dx"] = _exact_bwd_input(g, dout, k)
        outputs["dk"] = _exact_bwd_kernel(g, x, dout)
    return outputs
