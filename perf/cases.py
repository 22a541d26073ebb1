"""The work that a user of the integer-only inference library has it do, as measurable cases.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)` one more of the same ranges; `prepare`
makes what a program holds before the call (inputs, parameters, reordered weight copies, network handle, workspace) on the
GPU, `run` is one pass through the public entry points, `work` the bytes and operations that pass cannot do without.

Kinds of case
  forward        a whole ResNet18 / ResNet50 on one image batch (`hawq_forward_resnet`)
  conv           one quantised convolution layer, with or without a shortcut (`hawq_conv2d_int`)
  gemm           the fully connected layer / matrix product (`hawq_gemm_int`)
  residual_add   the stand-alone residual addition (`hawq_residual_add_dyadic`)
  module         an Inception-style module: requantised input, three convolutional branches, INT32 pooling branch,
                 concatenation (`hawq_conv2d_int`, `hawq_pool2d_sum_int`, `hawq_concat_dyadic`)
Every result is an integer with one correct value, so every comparison is exact.
"""
import math

import numpy as np
import torch

import paper_2011_10680_amd as hawq
import workloads as wl


# ---- cases ---------------------------------------------------------------------------------------------------------------

def _forward(name, arch, bits, batch, image=224, int32_shortcut=True):
    return dict(name=name, kind="forward", arch=arch, bits=bits, batch=batch, image=image, int32_shortcut=int32_shortcut)


def _conv(name, N, H, W, C, K, R, S, stride, pad, bits=8, shortcut=False):
    return dict(name=name, kind="conv", N=N, H=H, W=W, C=C, K=K, R=R, S=S, stride=stride, pad=pad, bits=bits, shortcut=shortcut)


def listed():
    return [
        # one image, one layer: the single-layer configuration of the benchmark, a pure latency measurement
        _conv("conv3x3_56x56x64_b1", 1, 56, 56, 64, 64, 3, 3, 1, 1),
        # a layer of the ResNet18-shaped 4-bit sweep at the batch the benchmark specifies
        _conv("conv3x3_14x14x256_int4_b8", 8, 14, 14, 256, 256, 3, 3, 1, 1, bits=4),
        # a down-sampling layer of the same sweep at its throughput batch
        _conv("conv3x3s2_56x56x64_128_b128", 128, 56, 56, 64, 128, 3, 3, 2, 1),
        # the closing layer of a bottleneck block with its shortcut, at a batch that fills no tile evenly
        _conv("conv1x1_28x28x128_512_shortcut_b37", 37, 28, 28, 128, 512, 1, 1, 1, 0, shortcut=True),
        # the classifier: pooled unsigned bytes to raw INT32 logits
        dict(name="gemm_fc_2048_1000_b128", kind="gemm", M=128, N=1000, K=2048, x="u8", y="s32"),
        # a residual addition on the INT32 accumulator of the main branch, stage-1 block output of 32 images
        dict(name="residual_add_56x56x256_b32", kind="residual_add", pixels=32 * 56 * 56, K=256, m="s32", r="u8", y="u8"),
        # the two Inception-style modules of tests and benchmark: a small one with ragged channel counts, a large one
        dict(name="module_17x17x64_b4", kind="module", N=4, H=17, C=64, bits=4),
        dict(name="module_35x35x288_b32", kind="module", N=32, H=35, C=288, bits=4),
        # interactive use: one image through the whole network
        _forward("resnet50_int8_b1", 50, "int8", 1),
        # the three whole-network workloads of the benchmark: ordinary, headline, largest (mixed precision)
        _forward("resnet18_int8_b64", 18, "int8", 64),
        _forward("resnet50_int8_b128", 50, "int8", 128),
        _forward("resnet50_mixed_b256", 50, "mixed", 256, int32_shortcut=False),
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["forward"] * 8 + ["conv"] * 7 + ["gemm"] * 2 + ["residual_add"] + ["module"] * 2)
    if kind == "forward":
        image = rng.choice([224, 224, 4 * rng.randrange(16, 81)])          # 64 .. 320 pixels
        most = max(1, min(256, int(240 * 224 * 224 / (image * image))))    # no more pixels than the largest listed case
        bits = rng.choice(["int8", "int8", "mixed", "int4"])
        return dict(kind="forward", arch=rng.choice([18, 50]), bits=bits, batch=_log_int(rng, 1, most), image=image,
                    int32_shortcut=bits == "int8" and rng.random() < 0.7)
    if kind == "conv":
        form = rng.choice(["3x3", "3x3", "3x3s2", "expand", "reduce", "1x1s2", "ragged"])
        bits = rng.choice([8, 8, 4])
        side = rng.choice([7, 14, 28, 56, rng.randrange(7, 57)])
        width = 64 * 56 // max(7, min(56, side))
        ch = min([64, 128, 256, 512], key=lambda c: abs(c - width))        # a ResNet's width at that resolution
        if form == "ragged":                                               # the windows and channel counts of Inception-style modules
            R, S = rng.choice([(1, 1), (3, 3), (5, 5), (5, 3)])
            side = rng.randrange(8, 36)
            C, K = 16 * rng.randrange(2, 19), 16 * rng.randrange(2, 19)
            shape = (side, side, C, K, R, S, 1, R // 2, False)
        elif form == "3x3":
            shape = (side, side, ch, ch, 3, 3, 1, 1, rng.random() < 0.3)
        elif form == "3x3s2":
            shape = (side, side, ch, 2 * ch, 3, 3, 2, 1, False)
        elif form == "1x1s2":
            shape = (side, side, 2 * ch, ch, 1, 1, 2, 0, False)
        elif form == "expand":
            shape = (side, side, ch, 4 * ch, 1, 1, 1, 0, True)
        else:
            shape = (side, side, 4 * ch, ch, 1, 1, 1, 0, False)
        H, W, C, K, R, S, stride, pad, shortcut = shape
        P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
        most = int(min(15e9 / (P * Q * K * R * S * C), 3e8 / (H * W * C), 3e8 / (P * Q * K)))
        c = _conv("", _log_int(rng, 1, max(1, min(128, most))), H, W, C, K, R, S, stride, pad, bits, shortcut)
        del c["name"]
        return c
    if kind == "gemm":
        y = rng.choice(["s32", "u8"])
        return dict(kind="gemm", M=_log_int(rng, 1, 4096), N=_log_int(rng, 10, 4096), K=64 * _log_int(rng, 4, 64), x=rng.choice(["u8", "s8"]), y=y)
    if kind == "residual_add":
        side, K = rng.choice([(56, 64), (56, 256), (28, 512), (14, 1024), (7, 2048)])
        return dict(kind="residual_add", pixels=_log_int(rng, 1, 64) * side * side, K=K, m=rng.choice(["s32", "s8"]),
                    r=rng.choice(["u8", "s8", "s32"]), y="u8")
    H = rng.choice([8, 17, 35, rng.randrange(8, 36)])
    return dict(kind="module", N=_log_int(rng, 1, max(1, min(64, 40000 // (H * H)))), H=H, C=rng.choice([64, 192, 256, 288]),
                bits=rng.choice([4, 8]))


# ---- inputs --------------------------------------------------------------------------------------------------------------

_HI = {8: 127, 4: 15}       # largest activation
_WM = {8: 127, 4: 7}        # largest weight
_X = {8: hawq.U8, 4: hawq.U4}
_WT = {8: hawq.S8, 4: hawq.S4}
_BYTES = {"s32": 4, "s8": 1, "u8": 1}
_DT = {"s32": hawq.S32, "s8": hawq.S8, "u8": hawq.U8}
_TD = {"s32": torch.int32, "s8": torch.int8, "u8": torch.uint8}


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed & 0x7fffffffffff)


def _ints(g, lo, hi, shape, dtype):
    """Uniform integers in [lo, hi]."""
    return torch.randint(lo, hi + 1, shape, dtype=dtype, device="cuda", generator=g)


def _packed(g, lo, hi, shape, bits, dtype):
    """A tensor of uniform integers in its stored form: bytes, or two 4-bit elements per byte along the last axis."""
    if bits == 8:
        return _ints(g, lo, hi, shape, dtype)
    half = tuple(shape[:-1]) + (shape[-1] // 2,)
    low, high = _ints(g, lo, hi, half, torch.int16), _ints(g, lo, hi, half, torch.int16)
    return ((low & 15) | ((high & 15) << 4)).to(torch.uint8)


def _dyadic(g, K, scale):
    """Per-channel multipliers b / 2^c around `scale`: b uniform in [2^14, 2^15), the shift with a 0 / 1 jitter."""
    c0 = int(math.floor(math.log2(1.5 * (1 << 14) / scale)))
    return _ints(g, 1 << 14, (1 << 15) - 1, (K,), torch.int32), _ints(g, c0, c0 + 1, (K,), torch.uint8)


def _layer(g, C, K, R, S, bits, m2):
    """Weights, bias and multipliers of a layer whose outputs spread over the clamp range; m2: E[x^2] of its input."""
    wm, hi = _WM[bits], _HI[bits]
    sigma = math.sqrt(R * S * C * m2 * wm * (wm + 1) / 3.0)
    w = _packed(g, -wm, wm, (K, R, S, C), bits, torch.int8)
    bias = ((torch.rand(K, device="cuda", generator=g) - 0.5) * sigma).round().to(torch.int32)
    b, c = _dyadic(g, K, hi / 3.0 / sigma)
    return dict(w=w, bias=bias, b=b, c=c, C=C, K=K, R=R, S=S)


def _conv_desc(N, H, W, L, stride, pad_h, pad_w, bits, y_dtype=None, raw=False):
    return hawq.ConvDesc(N=N, H=H, W=W, C=L["C"], K=L["K"], R=L["R"], S=L["S"], stride_h=stride, stride_w=stride, pad_h=pad_h, pad_w=pad_w,
                         x_dtype=_X[bits], w_dtype=_WT[bits], y_dtype=hawq.S32 if raw else (_X[bits] if y_dtype is None else y_dtype),
                         res_dtype=_X[bits], relu=0 if raw else 1, y_lo=-(1 << 31) if raw else 0, y_hi=(1 << 31) - 1 if raw else _HI[bits],
                         x_hi=127 if bits == 8 else 0)


def _weight_copies(desc, L):
    """The reordered weight copies the library offers for the layer, made once per layer and kept."""
    nb, nf = hawq.hawq_conv_blocked_weights_bytes(desc), hawq.hawq_conv_fragment_weights_bytes(desc)
    if nb:
        L["blocked"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
        hawq.hawq_conv_block_weights(desc, L["w"], L["blocked"])
        desc.w_blocked = L["blocked"].data_ptr()
    if nf:
        L["fragments"] = torch.empty(nf, dtype=torch.uint8, device="cuda")
        hawq.hawq_conv_fragment_weights(desc, L["w"], L["fragments"])
        desc.w_fragments = L["fragments"].data_ptr()
    return desc


def _bytes_of(K, bits):
    return K if bits == 8 else K // 2


def _prepare_forward(case, seed):
    if case["bits"] == "mixed":
        bits = wl.draw_bits(case["arch"], 4000 + case["arch"])
    elif case["bits"] == "int4":
        bits = {g: (8 if g in ("conv1", "fc") else 4) for g in wl.resnet_group_names(case["arch"])}
    else:
        bits = None
    net = wl.make_resnet(case["arch"], seed=seed, bits=bits, image_hw=case["image"], int32_shortcut=case["int32_shortcut"])
    handle = hawq.HawqNet(case["arch"], net["layers"], net["pool_b"], net["pool_c"], image_hw=case["image"])
    N = case["batch"]
    return dict(net=handle, N=N, x=_ints(_gen(seed), 0, 255, (N, case["image"], case["image"], 3), torch.uint8),
                logits=torch.empty((N, 1000), dtype=torch.int32, device="cuda"),
                workspace=torch.empty(handle.workspace_bytes(N), dtype=torch.uint8, device="cuda"))


def _prepare_conv(case, seed):
    g, bits, hi = _gen(seed), case["bits"], _HI[case["bits"]]
    N, H, W, C, K = case["N"], case["H"], case["W"], case["C"], case["K"]
    P, Q = (H + 2 * case["pad"] - case["R"]) // case["stride"] + 1, (W + 2 * case["pad"] - case["S"]) // case["stride"] + 1
    L = _layer(g, C, K, case["R"], case["S"], bits, hi * hi / 3.0)
    st = dict(L=L, x=_packed(g, 0, hi, (N, H, W, C), bits, torch.uint8),
              y=torch.empty((N, P, Q, _bytes_of(K, bits)), dtype=torch.uint8, device="cuda"), res=None, res_b=None, res_c=None)
    if case["shortcut"]:
        st["res"] = _packed(g, 0, hi, (N, P, Q, K), bits, torch.uint8)
        st["res_b"], st["res_c"] = _dyadic(g, K, 0.4)
    st["desc"] = _weight_copies(_conv_desc(N, H, W, L, case["stride"], case["pad"], case["pad"], bits), L)
    return st


def _prepare_gemm(case, seed):
    g = _gen(seed)
    M, N, K = case["M"], case["N"], case["K"]
    x = _ints(g, 0, 255, (M, K), torch.uint8) if case["x"] == "u8" else _ints(g, -128, 127, (M, K), torch.int8)
    sigma = math.sqrt(K * (255 * 255 / 3.0 if case["x"] == "u8" else 128 * 128 / 3.0) * 127 * 128 / 3.0)
    raw = case["y"] == "s32"
    b, c = (None, None) if raw else _dyadic(g, N, 42.0 / sigma)
    return dict(M=M, N=N, K=K, raw=raw, x=x, x_dt=_DT[case["x"]], y_dt=_DT[case["y"]], w=_ints(g, -127, 127, (N, K), torch.int8),
                bias=_ints(g, -(1 << 15), 1 << 15, (N,), torch.int32), b=b, c=c,
                y=torch.empty((M, N), dtype=_TD[case["y"]], device="cuda"))


def _prepare_residual_add(case, seed):
    g, P, K = _gen(seed), case["pixels"], case["K"]

    def branch(t):
        if t == "s32":     # an accumulator of about 18 bits
            return _ints(g, -(1 << 18), 1 << 18, (P, K), torch.int32), _dyadic(g, K, 2.0 ** -12)
        if t == "s8":
            return _ints(g, -128, 127, (P, K), torch.int8), _dyadic(g, K, 0.5)
        return _ints(g, 0, 127, (P, K), torch.uint8), _dyadic(g, K, 0.5)
    m, (mb, mc) = branch(case["m"])
    r, (rb, rc) = branch(case["r"])
    return dict(P=P, K=K, m=m, mb=mb, mc=mc, r=r, rb=rb, rc=rc, m_dt=_DT[case["m"]], r_dt=_DT[case["r"]], y_dt=_DT[case["y"]],
                y=torch.empty((P, K), dtype=torch.uint8, device="cuda"))


# (branch, layer, input, output channels, window); the last layer of a branch leaves its INT32 accumulator
_MODULE = [("b1", "b1", None, 64, 1), ("b2", "b2a", None, 48, 1), ("b2", "b2b", "b2a", 64, 3),
           ("b3", "b3a", None, 64, 1), ("b3", "b3b", "b3a", 96, 3), ("b3", "b3c", "b3b", 96, 3)]
_MODULE_OUT = ("b1", "b2b", "b3c")


def _prepare_module(case, seed):
    g, bits, N, H, C = _gen(seed), case["bits"], case["N"], case["H"], case["C"]
    hi, P = _HI[bits], N * H * H
    st = dict(N=N, H=H, C=C, P=P, x_dt=_X[bits], hi=hi, h=_ints(g, 0, (1 << 20) - 1, (N, H, H, C), torch.int32),
              rq=(torch.full((C,), 1 << 14, dtype=torch.int32, device="cuda"),
                  torch.full((C,), 34 - bits if bits == 4 else 27, dtype=torch.uint8, device="cuda")),
              low=torch.empty((P, _bytes_of(C, bits)), dtype=torch.uint8, device="cuda"), layers=[], cat=[])
    out = {}
    for _, name, src, K, R in _MODULE:
        raw = name in _MODULE_OUT
        Cin = C if src is None else out[src].shape[-1] * (8 // bits)
        m2 = hi * hi / 3.0
        L = _layer(g, Cin, K, R, R, bits, m2 if src is None else m2 * 0.4)
        L["sigma"] = math.sqrt(R * R * Cin * m2 * _WM[bits] * (_WM[bits] + 1) / 3.0)
        y = torch.empty((N, H, H, K if raw else _bytes_of(K, bits)), dtype=torch.int32 if raw else torch.uint8, device="cuda")
        d = _weight_copies(_conv_desc(N, H, H, L, 1, R // 2, R // 2, bits, raw=raw), L)
        st["layers"].append((d, st["low"] if src is None else out[src], L, raw, y))
        out[name] = y
        if raw:
            st["cat"].append((y, hawq.S32) + _dyadic(g, K, 60.0 / L["sigma"]))
    st["pool"] = torch.empty((N, H, H, C), dtype=torch.int32, device="cuda")
    st["cat"].append((st["pool"], hawq.S32) + _dyadic(g, C, 64.0 / (9 * (1 << 19))))
    st["y"] = torch.empty((P, 64 + 64 + 96 + C), dtype=torch.uint8, device="cuda")
    return st


def prepare(case, seed):
    st = dict(forward=_prepare_forward, conv=_prepare_conv, gemm=_prepare_gemm, residual_add=_prepare_residual_add,
              module=_prepare_module)[case["kind"]](case, seed)
    st["kind"] = case["kind"]
    return st


# ---- one pass ------------------------------------------------------------------------------------------------------------

def run(st):
    kind = st["kind"]
    if kind == "forward":
        st["net"].hawq_forward_resnet(st["x"], st["N"], st["logits"], st["workspace"])
        return st["logits"]
    if kind == "conv":
        L = st["L"]
        hawq.hawq_conv2d_int(st["desc"], st["x"], L["w"], L["bias"], L["b"], L["c"], st["res"], st["res_b"], st["res_c"], st["y"])
        return st["y"]
    if kind == "gemm":
        lo, hi = (-(1 << 31), (1 << 31) - 1) if st["raw"] else (0, 127)
        hawq.hawq_gemm_int(st["M"], st["N"], st["K"], st["x_dt"], hawq.S8, st["y_dt"], st["x"], st["w"], st["bias"], st["b"], st["c"],
                           0 if st["raw"] else 1, lo, hi, st["y"])
        return st["y"]
    if kind == "residual_add":
        hawq.hawq_residual_add_dyadic(st["P"], st["K"], st["m_dt"], st["r_dt"], st["y_dt"], st["m"], st["mb"], st["mc"], st["r"],
                                      st["rb"], st["rc"], 1, 0, 127, st["y"])
        return st["y"]
    # the INT32 feature map to low bits, the convolutional branches, the pooling branch on the map itself, the concatenation
    hawq.hawq_concat_dyadic(st["P"], [(st["h"], hawq.S32) + st["rq"]], st["x_dt"], 0, st["hi"], st["low"])
    for d, x, L, raw, y in st["layers"]:
        hawq.hawq_conv2d_int(d, x, L["w"], L["bias"], None if raw else L["b"], None if raw else L["c"], None, None, None, y)
    N, H, C = st["N"], st["H"], st["C"]
    hawq.hawq_pool2d_sum_int(N, H, H, C, 3, 3, 1, 1, 1, 1, hawq.S32, hawq.S32, st["h"], None, None, 0, 0, st["pool"])
    hawq.hawq_concat_dyadic(st["P"], st["cat"], hawq.U8, 0, 127, st["y"])
    return st["y"]


# ---- what a pass cannot do without ---------------------------------------------------------------------------------------

def _conv_work(N, H, W, C, K, R, S, P, Q, bits):
    sampled = P * Q if R * S == 1 else H * W      # a strided 1x1 reads only the sampled pixels
    return (N * sampled * C + K * R * S * C) * bits / 8.0 + 9.0 * K, 2.0 * N * P * Q * K * R * S * C


def work(case):
    kind = case["kind"]
    if kind == "forward":
        # image in, weights and parameters once, logits out: no activation between layers has to leave the chip
        N = case["batch"]
        bits = wl.draw_bits(case["arch"], 4000 + case["arch"]) if case["bits"] == "mixed" else None
        nbytes, flops = N * case["image"] ** 2 * 3 + 4.0 * N * 1000, 0.0
        for l in wl.resnet_layers(case["arch"], case["image"]):
            inner = l["group"] not in ("conv1", "fc")
            wbits = bits[l["group"]] if bits else (4 if case["bits"] == "int4" and inner else 8)
            macs = l["K"] * l["R"] * l["S"] * l["C"]
            nbytes += macs * wbits / 8.0 + 9.0 * l["K"]
            flops += 2.0 * N * l["P"] * l["Q"] * macs
        return dict(bytes=nbytes, flops=flops)
    if kind == "conv":
        N, H, W, K, bits = case["N"], case["H"], case["W"], case["K"], case["bits"]
        P, Q = (H + 2 * case["pad"] - case["R"]) // case["stride"] + 1, (W + 2 * case["pad"] - case["S"]) // case["stride"] + 1
        nbytes, flops = _conv_work(N, H, W, case["C"], K, case["R"], case["S"], P, Q, bits)
        out = N * P * Q * K * bits / 8.0
        return dict(bytes=nbytes + out * (2 if case["shortcut"] else 1) + (5.0 * K if case["shortcut"] else 0.0), flops=flops)
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return dict(bytes=float(M * K + N * K + M * N * _BYTES[case["y"]] + 9 * N), flops=2.0 * M * N * K)
    if kind == "residual_add":
        n = case["pixels"] * case["K"]
        return dict(bytes=float(n * (_BYTES[case["m"]] + _BYTES[case["r"]] + _BYTES[case["y"]]) + 10 * case["K"]), flops=8.0 * n)
    # the module: the INT32 map in, the concatenated bytes out, weights once
    N, H, C, bits = case["N"], case["H"], case["C"], case["bits"]
    P, widths = N * H * H, {None: C}
    nbytes, flops = P * C * 4.0 + P * (224 + C), 9.0 * P * C
    for _, name, src, K, R in _MODULE:
        widths[name] = K
        nbytes += K * R * R * widths[src] * bits / 8.0 + 9.0 * K
        flops += 2.0 * P * K * R * R * widths[src]
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    return "exact"
