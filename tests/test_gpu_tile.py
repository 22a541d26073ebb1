"""GPU parity of the tiled kernel with channels along the lanes: ragged channel counts, unsigned bytes above 127, INT32 results,
identity shortcuts, a second convolution, at the edges of every tile it chooses from, bit-exact."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hawq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as h
    h.load_library()
    return h


# (M, N, K): 64x32 tiles; 64x64 with a remainder in every direction and 1, 5 and 6 steps of the four-deep ring; 128x64; 128x128;
# 256x256; N % 4 of 0 .. 3; one row past a tile
_PRODUCTS = [(300, 1003, 1024), (769, 1002, 64), (1030, 1001, 320), (1025, 1000, 384), (3000, 301, 192), (4099, 999, 768), (4097, 1004, 256),
             (2100, 4002, 1024)]


@pytest.mark.parametrize("M,N,K", _PRODUCTS)
@pytest.mark.parametrize("x_dt,y_dt", [(oracle.U8, oracle.S32), (oracle.S8, oracle.S32), (oracle.U8, oracle.U8), (oracle.S8, oracle.S8)])
def test_matrix_product(hawq, M, N, K, x_dt, y_dt):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(M + N + K)
    x = g.integers(0, 256, size=(M, K)).astype(np.uint8) if x_dt == oracle.U8 else g.integers(-128, 128, size=(M, K)).astype(np.int8)
    w = g.integers(-127, 128, size=(N, K)).astype(np.int8)
    w[0], w[N - 1] = -128, 127
    bias = g.integers(-(1 << 15), 1 << 15, size=N).astype(np.int32)
    raw = y_dt == oracle.S32
    b = c = None
    if not raw:
        s = np.sqrt(K) * 74 * (148 if x_dt == oracle.U8 else 74) / 42
        b = g.integers(1 << 14, 1 << 15, size=N).astype(np.int32)
        c = (int(np.log2(1.5 * (1 << 14) * s)) + g.integers(0, 2, size=N)).astype(np.uint8)
    lo, hi = (0, 0) if raw else {oracle.U8: (0, 255), oracle.S8: (-128, 127)}[y_dt]
    y = torch.full((M, N), 0x5A, dtype={oracle.U8: torch.uint8, oracle.S8: torch.int8, oracle.S32: torch.int32}[y_dt], device="cuda")
    hawq.hawq_gemm_int(M, N, K, x_dt, hawq.S8, y_dt, to_dev(x), to_dev(w), to_dev(bias), to_dev(b), to_dev(c), 0, lo, hi, y)
    torch.cuda.synchronize()
    want = oracle.conv2d_int(x.reshape(1, 1, M, K), w, bias, b, c, N=1, H=1, W=M, C=K, K=N, R=1, S=1, stride=1, pad=0, x_dt=x_dt, w_dt=oracle.S8,
                             y_dt=y_dt, relu=0, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy(), np.asarray(want).reshape(M, N), str((M, N, K)))


# (N, H, W, C, K, R, S, stride, pad, bits, what): windows and channel counts whose 64-byte steps hold several taps, or parts of them;
# what: "raw", "wide" (one channel outside the narrow evaluation's range), "byte" (unsigned bytes above 127), "s" (signed result)
_WINDOWS = [
    (9, 35, 34, 96, 96, 3, 3, 1, 1, 8, ""), (9, 35, 34, 96, 97, 3, 3, 1, 1, 8, "raw"), (8, 34, 33, 112, 90, 3, 3, 1, 1, 8, "wide"),
    (23, 35, 35, 16, 32, 5, 3, 1, 2, 8, "raw"), (30, 41, 39, 48, 66, 3, 3, 2, 1, 8, "s"), (14, 33, 35, 64, 80, 3, 3, 1, 1, 8, ""),
    (9, 35, 34, 80, 96, 3, 3, 1, 1, 8, "byte"), (12, 61, 60, 144, 275, 1, 1, 2, 0, 8, "byte"),
    (13, 35, 35, 288, 64, 1, 1, 1, 0, 4, "raw"), (13, 35, 35, 288, 70, 1, 1, 1, 0, 4, ""), (9, 35, 34, 96, 100, 3, 3, 1, 1, 4, ""),
    (15, 35, 33, 32, 62, 5, 5, 1, 2, 4, "s"), (9, 35, 34, 160, 98, 3, 3, 1, 1, 4, "wide"), (14, 33, 35, 128, 96, 3, 3, 1, 1, 4, ""),
    (40, 35, 35, 224, 300, 1, 1, 1, 0, 4, ""),
]


@pytest.mark.parametrize("shape", _WINDOWS)
def test_convolution_windows(hawq, shape):
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    N, H, W, C, K, R, S, stride, pad, bits, what = shape
    case = _scale_c(wl.conv_case(seed=sum(shape[:10]), N=N, H=H, W=W, C=C, K=K, R=R, S=S, stride=stride, pad=pad, bits=bits), bits)
    if what == "byte":
        case["x"] = np.random.default_rng(K).integers(0, 256, size=case["x"].shape).astype(np.uint8)
        case["c"] = case["c"] + np.uint8(1)
    if what == "wide":
        case["b"][K // 2], case["c"][K // 2] = (1 << 31) - 1, case["c"][K // 2] + 16
    if bits == 4:
        wu = oracle.unpack(case["w"], oracle.S4).reshape(K, R, S, C)
        wu[0], wu[K - 1] = -8, 7
        case["w"] = wl.pack_nibbles(wu).reshape(case["w"].shape)
    raw = what == "raw"
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    y_dt = hawq.S32 if raw else {(8, True): hawq.S8, (8, False): hawq.U8, (4, True): hawq.S4, (4, False): hawq.U4}[bits, what == "s"]
    lo, hi = {(8, True): (-128, 127), (8, False): (0, 127), (4, True): (-8, 7), (4, False): (0, 15)}[bits, what == "s"]
    got, want = run_conv_gpu(case, x_dt, w_dt, y_dt, y_lo=lo, y_hi=hi, raw=raw, relu=0 if raw or what == "s" else 1, x_hi=127 if bits == 8 and what != "byte" else 0)
    assert_same(got, want, str(shape))
    if not raw:
        v = want.astype(np.int32) if bits == 8 else oracle.unpack(want, y_dt)
        assert len(np.unique(v)) > 8


def test_blocked_weights(hawq):
    """The blocked copy in place of the weights' rows, whole and ragged channel tiles."""
    import torch
    from gpu_util import to_dev, assert_same
    from test_gpu_conv import _scale_c
    for bits, C, K in ((8, 192, 96), (4, 128, 100)):
        case = _scale_c(wl.conv_case(seed=K, N=9, H=35, W=34, C=C, K=K, R=3, S=3, stride=1, pad=1, bits=bits), bits)
        x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
        d = hawq.ConvDesc(N=9, H=35, W=34, C=C, K=K, R=3, S=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, x_dtype=x_dt, w_dtype=w_dt,
                          y_dtype=x_dt, res_dtype=hawq.U8, relu=1, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
        w = to_dev(case["w"])
        blocked = torch.empty(hawq.hawq_conv_blocked_weights_bytes(d), dtype=torch.uint8, device="cuda")
        hawq.hawq_conv_block_weights(d, w, blocked)
        d.w_blocked = blocked.data_ptr()
        y = torch.full((9, 35, 34, K * bits // 8), 0x5A, dtype=torch.uint8, device="cuda")
        hawq.hawq_conv2d_int(d, to_dev(case["x"]), w, to_dev(case["bias"]), to_dev(case["b"]), to_dev(case["c"]), None, None, None, y)
        torch.cuda.synchronize()
        want = oracle.conv2d_int(case["x"], case["w"], case["bias"], case["b"], case["c"], N=9, H=35, W=34, C=C, K=K, R=3, S=3, stride=1, pad=1,
                                 x_dt=x_dt, w_dt=w_dt, y_dt=x_dt, relu=1, y_lo=0, y_hi=hi)
        assert_same(y.cpu().numpy(), want, str((bits, C, K)))


def _tile(M, C, K, R, bits):
    """The tile of a launch without a shortcut (tile_choice and few_tiles of csrc/conv_tile.hip)."""
    steps = (R * R * C * bits // 8 + 63) // 64
    costs = []
    for bm, bn, chain in ((256, 256, 75), (128, 128, 37), (128, 64, 27), (64, 64, 20), (64, 32, 17)):
        per_cu = (-(-M // bm) * -(-K // bn) + 255) // 256
        costs.append((steps * max(per_cu * (bm + bn) * 64 // 512, chain) + per_cu * bm * bn // 150, len(costs)))
    best = min(costs)[1]
    if best < 3 and -(-M // 64) * -(-K // 64) <= (768 if steps < 16 else 512 if steps < 32 else 0):
        best = 3
    return ((256, 256), (128, 128), (128, 64), (64, 64), (64, 32))[best]


# the larger tiles over windows, several steps and one, ragged in pixels and channels: (N, H, W, C, K, R, bits, what, tile, blocked weights)
_LARGE = [
    (1, 223, 222, 48, 33, 3, 8, "", (128, 64), False), (1, 223, 222, 16, 34, 5, 8, "byte", (128, 64), False), (3, 129, 131, 96, 35, 3, 4, "", (128, 64), False),
    (1, 159, 161, 80, 97, 3, 8, "", (128, 128), False), (1, 159, 161, 112, 99, 3, 8, "byte", (128, 128), False), (1, 201, 201, 160, 97, 3, 4, "", (128, 128), False),
    (2, 113, 115, 16, 67, 5, 8, "s", (128, 128), False), (1, 159, 161, 64, 97, 3, 8, "", (128, 128), True), (1, 201, 203, 128, 97, 3, 4, "", (128, 128), True),
    (1, 235, 237, 48, 161, 3, 8, "", (256, 256), False), (1, 183, 182, 48, 194, 5, 8, "byte", (256, 256), False), (1, 245, 245, 32, 163, 5, 4, "", (256, 256), False),
    (1, 235, 237, 96, 161, 3, 4, "s", (256, 256), False), (1, 235, 237, 64, 161, 3, 8, "", (256, 256), True), (1, 245, 243, 128, 163, 3, 4, "", (256, 256), True),
]


@pytest.mark.parametrize("shape", _LARGE)
def test_large_tiles_over_windows(hawq, shape):
    import torch
    from gpu_util import to_dev, assert_same
    from test_gpu_conv import _scale_c
    N, H, W, C, K, R, bits, what, tile, block = shape
    assert _tile(N * H * W, C, K, R, bits) == tile
    case = _scale_c(wl.conv_case(seed=sum(shape[:7]), N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, bits=bits), bits)
    if what == "byte":
        case["x"] = np.random.default_rng(K).integers(0, 256, size=case["x"].shape).astype(np.uint8)
        case["c"] = case["c"] + np.uint8(1)
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    y_dt = {(8, True): hawq.S8, (8, False): hawq.U8, (4, True): hawq.S8, (4, False): hawq.U8}[bits, what == "s"]
    lo, hi, relu = (-128, 127, 0) if what == "s" else (0, 127, 1)
    d = hawq.ConvDesc(N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride_h=1, stride_w=1, pad_h=R // 2, pad_w=R // 2, x_dtype=x_dt, w_dtype=w_dt,
                      y_dtype=y_dt, res_dtype=hawq.U8, relu=relu, y_lo=lo, y_hi=hi, x_hi=127 if bits == 8 and what != "byte" else 0)
    w = to_dev(case["w"])
    if block:
        blocked = torch.empty(hawq.hawq_conv_blocked_weights_bytes(d), dtype=torch.uint8, device="cuda")
        hawq.hawq_conv_block_weights(d, w, blocked)
        d.w_blocked = blocked.data_ptr()
    y = torch.full((N, H, W, K), 0x5A, dtype=torch.uint8, device="cuda")
    hawq.hawq_conv2d_int(d, to_dev(case["x"]), w, to_dev(case["bias"]), to_dev(case["b"]), to_dev(case["c"]), None, None, None, y)
    torch.cuda.synchronize()
    want = oracle.conv2d_int(case["x"], case["w"], case["bias"], case["b"], case["c"], N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride=1, pad=R // 2,
                             x_dt=x_dt, w_dt=w_dt, y_dt=y_dt, relu=relu, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy().view(want.dtype), want, str(shape))
    assert len(np.unique(want)) > 8


# (N, H, W, C, K, R, stride, bits, shortcut's type, what): 64x64 tiles with remainders in pixels and channels, one K-step and
# many, channel counts of 4, 8 and 12 past a group of 16, results of either sign and width; what: "wide" (one channel's main and
# another's shortcut parameters outside the narrow evaluation's range), "s" (signed result)
_SHORTCUTS = [
    (1, 56, 56, 64, 256, 1, 1, 8, oracle.U8, ""), (1, 56, 55, 64, 256, 1, 1, 8, oracle.S8, "wide"), (7, 29, 31, 128, 128, 3, 1, 8, oracle.U8, "s"),
    (16, 35, 34, 96, 68, 1, 1, 8, oracle.U8, "wide"), (9, 33, 33, 48, 84, 3, 1, 8, oracle.S8, ""), (14, 33, 35, 80, 44, 1, 1, 8, oracle.U4, ""),
    (1, 56, 56, 64, 256, 1, 1, 4, oracle.U4, ""), (5, 56, 55, 64, 64, 3, 1, 4, oracle.U4, "wide"), (12, 14, 14, 256, 256, 3, 1, 4, oracle.U8, ""),
    (24, 35, 35, 96, 76, 1, 1, 4, oracle.S8, "s"), (20, 35, 35, 96, 92, 3, 2, 4, oracle.U4, "s"),
]


@pytest.mark.parametrize("shape", _SHORTCUTS)
def test_identity_shortcut(hawq, shape):
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    N, H, W, C, K, R, stride, bits, res_dt, what = shape
    case = _scale_c(wl.conv_case(seed=sum(shape[:8]), N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride=stride, pad=R // 2, bits=bits), bits)
    g = np.random.default_rng(K + N)
    P, Q = (H + 2 * (R // 2) - R) // stride + 1, (W + 2 * (R // 2) - R) // stride + 1
    rl, rh = {oracle.U8: (0, 255), oracle.S8: (-128, 127), oracle.U4: (0, 15)}[res_dt]
    res = g.integers(rl, rh + 1, size=(N, P, Q, K))
    case["residual"] = wl.pack_nibbles(res) if res_dt == oracle.U4 else res.astype(np.int8 if res_dt == oracle.S8 else np.uint8)
    # a shortcut of about the range of the result: rescaled by 1/2 .. 1 (8-bit results), to a quarter of that for packed ones
    case["res_b"] = g.integers(1 << 14, 1 << 15, size=K).astype(np.int32)
    case["res_c"] = np.full(K, {(8, oracle.U4): 12, (4, oracle.U8): 19, (4, oracle.S8): 19}.get((bits, res_dt), 15), np.uint8)
    if what == "wide":
        case["b"][K // 2], case["c"][K // 2] = (1 << 31) - 1, case["c"][K // 2] + 16
        case["res_b"][1], case["res_c"][1] = (1 << 31) - 1, 31
    signed = what == "s"
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    y_dt = {(8, True): hawq.S8, (8, False): hawq.U8, (4, True): hawq.S4, (4, False): hawq.U4}[bits, signed]
    lo, hi = {(8, True): (-128, 127), (8, False): (0, 255), (4, True): (-8, 7), (4, False): (0, 15)}[bits, signed]
    got, want = run_conv_gpu(case, x_dt, w_dt, y_dt, res_dt=res_dt, y_lo=lo, y_hi=hi, relu=0 if signed else 1, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str(shape))
    v = want.astype(np.int32) if bits == 8 else oracle.unpack(want, y_dt)
    assert len(np.unique(v)) > 8


# (N, H, C, K, R, Cs, stride of the shortcut, bits, wide, result): one and several steps of either branch, remainders in pixels and
# channels, chunks that end within a step, signed results
_DUAL = [
    (1, 56, 64, 256, 1, 64, 1, 8, False, oracle.U8), (3, 28, 128, 512, 1, 256, 2, 8, True, oracle.U8), (7, 28, 128, 128, 3, 64, 2, 8, False, oracle.S8),
    (9, 23, 80, 116, 1, 48, 2, 8, False, oracle.U8), (9, 31, 48, 84, 3, 16, 1, 8, True, oracle.U4), (1, 56, 64, 256, 1, 64, 1, 4, False, oracle.U4),
    (2, 14, 256, 1024, 1, 512, 2, 4, True, oracle.U4), (2, 5, 32, 36, 1, 32, 2, 4, False, oracle.U8), (3, 17, 96, 76, 3, 160, 2, 4, True, oracle.S4),
]


@pytest.mark.parametrize("shape", _DUAL)
def test_two_convolutions(hawq, shape):
    from gpu_util import assert_same
    from test_gpu_dual import _case, _run
    N, H, C, K, R, Cs, ss, bits, wide, y_dt = shape
    t = _case(sum(shape[:8]), N, H, C, K, R, Cs, ss, bits=bits, wide=wide)
    lo, hi = {oracle.U8: (0, 255), oracle.S8: (-128, 127), oracle.U4: (0, 15), oracle.S4: (-8, 7)}[y_dt]
    got, want = _run(hawq, t, y_dt, 0 if lo else 1, lo, hi)
    assert_same(got, want, str(shape))
    v = want.astype(np.int32) if y_dt in (oracle.U8, oracle.S8) else oracle.unpack(want, y_dt)
    assert len(np.unique(v)) > 8


# two convolutions that the kernel of whole 64-channel steps does not take, either side of the lines to the split-reduction kernel
# (a 64 x 64 tile per CU with a step more than this kernel takes there, one fewer, more tiles) and that kernel's 64-channel tiles
@pytest.mark.parametrize("N,H,C,K,R,Cs,ss", [(1, 32, 256, 1020, 1, 1024, 1), (1, 32, 320, 1020, 1, 1024, 1), (1, 33, 320, 1020, 1, 1024, 1),
                                             (1, 56, 128, 1024, 3, 48, 2), (1, 56, 336, 256, 1, 1024, 2)])
def test_two_convolutions_at_the_lines(hawq, N, H, C, K, R, Cs, ss):
    test_two_convolutions(hawq, (N, H, C, K, R, Cs, ss, 8, False, oracle.U8))


# (pixels, C, K, R, bits, shortcut): either side of the lines between this kernel, the split-reduction kernel and the one with pixels along
# the lanes: packed operands with a 32 x 64 tile per CU and one more; packed windows with a 64 x 64 tile per CU and one more, with
# and without a shortcut; narrow shortcuts; a long reduction over few channels; a shortcut of fewer than 1024 pixels; the split-reduction
# kernel's small tiles (one round and its end, two) and whole 64 channels
_LINES = [
    ((52, 64), 448, 148, 1, 4, False), ((52, 63), 448, 148, 1, 4, False), ((49, 64), 224, 320, 3, 4, False), ((49, 84), 224, 256, 3, 4, False),
    ((41, 64), 96, 384, 3, 4, True), ((43, 65), 96, 384, 3, 4, True), ((201, 177), 192, 16, 3, 4, True), ((201, 220), 192, 12, 3, 8, True),
    ((181, 193), 464, 12, 3, 8, False), ((397, 247), 432, 12, 3, 8, False), ((31, 33), 384, 512, 3, 4, True), ((31, 33), 192, 512, 3, 8, True), ((136, 64), 544, 36, 1, 8, True),
    ((137, 64), 544, 36, 1, 8, True), ((255, 64), 96, 32, 3, 8, False),
]


@pytest.mark.parametrize("shape", _LINES)
def test_lines_of_the_dispatch(hawq, shape):
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    (H, W), C, K, R, bits, res = shape
    case = _scale_c(wl.conv_case(seed=H + W + C + K, N=1, H=H, W=W, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, bits=bits, with_residual=res), bits)
    x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
    got, want = run_conv_gpu(case, x_dt, w_dt, x_dt, res_dt=x_dt, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str(shape))
