"""GPU parity of the split-reduction kernel: small launches and channel counts that are only a multiple of 16, bit-exact."""
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


# (N, H, W, C, K, R, S, stride, pad, bits, shortcut, raw): every tile shape with whole and ragged tiles, reductions of one
# step, of fewer steps than waves, of exactly a ring and of a ring and a remainder, taps that split a 64-byte step
_SHAPES = [
    (1, 4, 4, 16, 16, 1, 1, 1, 0, 8, False, False),       # 16x16, a quarter of one step
    (1, 5, 7, 48, 36, 3, 3, 1, 1, 8, True, False),        # 16x16, K % 16 != 0, shortcut
    (1, 7, 7, 512, 512, 3, 3, 1, 1, 8, False, False),     # 16x16, nine steps per wave: a ring of eight and one
    (2, 14, 14, 256, 272, 3, 3, 1, 1, 8, True, False),    # 16x32 / 32x32
    (3, 14, 13, 80, 208, 5, 3, 1, 2, 8, False, True),     # 5x3 window, INT32 output
    (4, 7, 7, 2048, 512, 1, 1, 1, 0, 8, False, False),    # long pointwise reduction
    (5, 28, 28, 144, 96, 3, 3, 2, 1, 8, False, False),    # strided, 32x64 of few steps
    (16, 7, 7, 576, 512, 3, 3, 1, 1, 8, False, False),    # 32x64 over eight waves
    (9, 28, 27, 112, 80, 1, 1, 1, 0, 8, True, False),     # 64x64
    (22, 35, 35, 96, 96, 3, 3, 1, 1, 8, False, False),    # past one round, last channel tile half empty: 32x128
    (24, 33, 35, 48, 128, 3, 3, 1, 1, 8, False, True),    # past one round: 64x128
    (1, 3, 3, 64, 7, 3, 3, 1, 1, 8, False, False),        # K % 4 != 0: element-wise epilogue
    (2, 9, 9, 32, 18, 3, 3, 1, 1, 4, True, False),        # packed, 16-byte chunks, K % 4 != 0
    (2, 9, 11, 48, 64, 3, 3, 1, 1, 4, False, False),      # packed, 8-byte chunks
    (1, 14, 14, 256, 256, 3, 3, 1, 1, 4, False, True),    # packed, whole 128-channel steps, INT32 output
    (4, 17, 17, 96, 96, 3, 3, 1, 1, 4, False, False),     # packed, a step spans two taps
    (24, 35, 35, 288, 64, 1, 1, 1, 0, 4, False, True),    # packed, 64x128
    (24, 35, 35, 48, 96, 3, 3, 1, 1, 4, True, False),     # packed, 8-byte chunks, 32x128
]


@pytest.mark.parametrize("shape", _SHAPES)
def test_split_reduction_shapes(hawq, shape):
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    N, H, W, C, K, R, S, stride, pad, bits, res, raw = shape
    case = _scale_c(wl.conv_case(seed=sum(shape[:10]), N=N, H=H, W=W, C=C, K=K, R=R, S=S, stride=stride, pad=pad, bits=bits,
                                 with_residual=res), bits)
    if bits == 4:      # the extremes of the signed weights next to the largest activation
        wu = oracle.unpack(case["w"], oracle.S4).reshape(K, R, S, C)
        wu[0], wu[K - 1] = -8, 7
        case["w"] = wl.pack_nibbles(wu).reshape(case["w"].shape)
    x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
    got, want = run_conv_gpu(case, x_dt, w_dt, hawq.S32 if raw else x_dt, res_dt=x_dt, y_lo=0, y_hi=hi, raw=raw,
                             relu=0 if raw else 1, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str(shape))
    if not raw:
        v = want.astype(np.int32) if bits == 8 else oracle.unpack(want, oracle.U4)
        assert 0.02 < (v > 0).mean() and len(np.unique(v)) > 5


@pytest.mark.parametrize("C", [(1 << 20) - 32, 1 << 20, 1200000])
def test_longest_packed_reductions(hawq, C):
    """Sums of all-extreme packed operands on both sides of the length up to which sixteen times a sum fits 32 bits."""
    from gpu_util import run_conv_gpu, assert_same
    case = wl.conv_case(seed=5, N=1, H=1, W=1, C=32, K=16, R=1, S=1, stride=1, pad=0, bits=4)
    case["C"] = C
    case["x"] = np.full(case["x"].shape[:-1] + (C // 2,), 0xFF, dtype=case["x"].dtype)                    # 15
    case["w"] = np.full(case["w"].shape[:-1] + (C // 2,), 0x88, dtype=np.uint8).view(case["w"].dtype)     # -8
    got, want = run_conv_gpu(case, hawq.U4, hawq.S4, hawq.S32, raw=True, x_hi=0, y_lo=0, y_hi=0, relu=0)
    assert_same(got, want, str(C))
    assert (np.abs(want.astype(np.int64) + 120 * C) < 1 << 28).all()


@pytest.mark.parametrize("N,H,C,K,R,pad", [(2, 9, 64, 48, 3, 1), (24, 20, 176, 272, 3, 1), (3, 8, 16, 16, 1, 0)])
def test_unsigned_bytes_over_the_whole_range_with_padding(hawq, N, H, C, K, R, pad):
    """x - 128 on the matrix cores: padding taps and the chunks past the reduction's end must cancel exactly."""
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + C, N=N, H=H, W=H, C=C, K=K, R=R, S=R, stride=1, pad=pad, bits=8), 8)
    case["x"] = np.random.default_rng(C).integers(0, 256, size=case["x"].shape, dtype=np.uint8)
    got, want = run_conv_gpu(case, hawq.U8, hawq.S8, hawq.S32, raw=True, x_hi=0, y_lo=0, y_hi=0, relu=0)
    assert_same(got, want)


@pytest.mark.parametrize("M,N,K,x_signed,raw", [(1, 10, 256, False, True), (16, 1000, 512, False, True), (237, 551, 384, False, False),
                                                (820, 323, 576, False, False), (2865, 33, 320, True, False), (4096, 200, 1024, False, True)])
def test_gemm_any_size(hawq, M, N, K, x_signed, raw):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(M + N + K)
    x = g.integers(-128, 128, size=(M, K)).astype(np.int8) if x_signed else g.integers(0, 256, size=(M, K), dtype=np.uint8)
    w = g.integers(-127, 128, size=(N, K)).astype(np.int8)
    bias = g.integers(-(1 << 15), 1 << 15, size=N).astype(np.int32)
    b = g.integers(1 << 14, 1 << 15, size=N).astype(np.int32)
    c = np.full(N, 15 + int(np.ceil(np.log2(K * 40.0))), dtype=np.uint8)
    x_dt = hawq.S8 if x_signed else hawq.U8
    y = torch.full((M, N), 0x5A, dtype=torch.int32 if raw else torch.uint8, device="cuda")
    hawq.hawq_gemm_int(M, N, K, x_dt, hawq.S8, hawq.S32 if raw else hawq.U8, to_dev(x), to_dev(w), to_dev(bias), None if raw else to_dev(b),
                       None if raw else to_dev(c), 0 if raw else 1, 0, 0 if raw else 127, y)
    torch.cuda.synchronize()
    want = oracle.gemm_int(x, w, bias, None if raw else b, None if raw else c, M=M, N=N, K=K, x_dt=x_dt, w_dt=oracle.S8,
                           y_dt=oracle.S32 if raw else oracle.U8, relu=0 if raw else 1, y_lo=0, y_hi=127)
    assert_same(y.cpu().numpy(), want)


@pytest.mark.parametrize("N,H,C,K,R,Hs,Cs,stride_s", [(1, 7, 512, 2048, 1, 14, 1024, 2), (1, 14, 256, 256, 3, 28, 128, 2), (3, 8, 80, 96, 3, 8, 48, 1),
                                                      (2, 7, 64, 72, 1, 13, 64, 2)])
def test_two_convolutions_split_reduction(hawq, N, H, C, K, R, Hs, Cs, stride_s):
    """Block output with a convolution on both branches: the waves are divided between the two reductions."""
    import torch
    from gpu_util import to_dev, assert_same
    from test_gpu_conv import _scale_c
    m = _scale_c(wl.conv_case(seed=C + K, N=N, H=H, W=H, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, bits=8), 8)
    s = _scale_c(wl.conv_case(seed=C + K + 1, N=N, H=Hs, W=Hs, C=Cs, K=K, R=1, S=1, stride=stride_s, pad=0, bits=8), 8)
    assert (m["P"], m["Q"]) == (s["P"], s["Q"])

    def desc(c):
        return hawq.ConvDesc(N=c["N"], H=c["H"], W=c["W"], C=c["C"], K=K, R=c["R"], S=c["S"], stride_h=c["stride"], stride_w=c["stride"],
                             pad_h=c["pad"], pad_w=c["pad"], x_dtype=hawq.U8, w_dtype=hawq.S8, y_dtype=hawq.U8, res_dtype=hawq.U8, relu=1,
                             y_lo=0, y_hi=127, x_hi=127)
    y = torch.full((N, m["P"], m["Q"], K), 0x5A, dtype=torch.uint8, device="cuda")
    p = lambda c: [to_dev(c[k]) for k in ("x", "w", "bias", "b", "c")]
    hawq.hawq_conv2d_dual_int(desc(m), *p(m), desc(s), *p(s), y)
    torch.cuda.synchronize()
    want = oracle.conv2d_dual_int(m["x"], m["w"], m["bias"], m["b"], m["c"], s["x"], s["w"], s["bias"], s["b"], s["c"],
                                  N=N, H=H, W=H, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, Hs=Hs, Ws=Hs, Cs=Cs, Rs=1, Ss=1, stride_s=stride_s, pad_s=0,
                                  x_dt=oracle.U8, w_dt=oracle.S8, xs_dt=oracle.U8, ws_dt=oracle.S8, y_dt=oracle.U8, relu=1, y_lo=0, y_hi=127)
    assert_same(y.cpu().numpy(), want)
