"""GPU parity of the whole-row 3x3 kernel for 64 input channels (stride 1 and 2), bit-exact: tiles of several heights with
ragged last tiles and column tiles, odd image sizes, both channel splits, shortcuts, packed operands and outputs, parameters
outside the narrow evaluation."""
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


@pytest.mark.parametrize("N,H,W,K,stride,bits,res,y4", [
    (17, 56, 56, 64, 1, 8, 0, False), (23, 47, 49, 64, 1, 8, None, True), (6, 93, 101, 128, 1, 8, 1, False), (61, 30, 31, 64, 1, 8, 2, True),
    (200, 16, 17, 64, 1, 8, None, False), (5, 112, 111, 64, 1, 4, 2, True),
    (17, 56, 56, 128, 2, 8, None, False), (19, 55, 57, 64, 2, 8, 0, False), (31, 45, 63, 192, 2, 8, None, True), (64, 56, 56, 128, 2, 4, None, True),
])
def test_whole_rows_64_channels(hawq, N, H, W, K, stride, bits, res, y4):
    import torch
    from gpu_util import to_dev, out_shape, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + W + K, N=N, H=H, W=W, C=64, K=K, R=3, S=3, stride=stride, pad=1, bits=bits,
                                 with_residual=res is not None, res_signed=res == 1), bits)
    if res == 2 and bits == 8:
        case["residual"] = wl.pack_nibbles(np.random.default_rng(K).integers(0, 16, size=case["residual"].shape))
    if y4 and bits == 8:
        case["c"] = (case["c"] + 3).astype(np.uint8)
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    y_dt, hi = (hawq.U4, 15) if y4 else (hawq.U8, 127)
    P, Q = case["P"], case["Q"]
    d = hawq.ConvDesc(N=N, H=H, W=W, C=64, K=K, R=3, S=3, stride_h=stride, stride_w=stride, pad_h=1, pad_w=1, x_dtype=x_dt, w_dtype=w_dt,
                      y_dtype=y_dt, res_dtype=res or 0, relu=1, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
    w = to_dev(case["w"])
    wf = torch.empty(hawq.hawq_conv_fragment_weights_bytes(d), dtype=torch.uint8, device="cuda")
    hawq.hawq_conv_fragment_weights(d, w, wf)
    d.w_fragments = wf.data_ptr()
    for wide in (False, True):
        b, c = case["b"], case["c"]
        if wide:
            b, c = (b.astype(np.int64) << 14).astype(np.int32), (c.astype(np.int32) + 14).astype(np.uint8)
        y = torch.full(out_shape((N, P, Q, K), y_dt), 0x5A, dtype=torch.uint8, device="cuda")
        r = [to_dev(case[k]) if res is not None else None for k in ("residual", "res_b", "res_c")]
        hawq.hawq_conv2d_int(d, to_dev(case["x"]), w, to_dev(case["bias"]), to_dev(b), to_dev(c), *r, y)
        torch.cuda.synchronize()
        want = oracle.conv2d_int(case["x"], case["w"], case["bias"], b, c, N=N, H=H, W=W, C=64, K=K, R=3, S=3, stride=stride, pad=1,
                                 x_dt=x_dt, w_dt=w_dt, y_dt=y_dt, relu=1, y_lo=0, y_hi=hi, residual=case.get("residual") if res is not None else None,
                                 res_b=case.get("res_b"), res_c=case.get("res_c"), res_dt=res or 0)
        assert_same(y.cpu().numpy(), want, str((N, H, W, K, stride, bits, wide)))
    v = oracle.unpack(want, oracle.U4) if y4 else want.astype(np.int32)
    assert 0.02 < (v > 0).mean() and (v == hi).mean() < 0.7


@pytest.mark.parametrize("N,H,W,K,stride,bits,res,y4", [
    # 64 -> 64 up to 62 columns: with a shortcut past 65536 pixels; column tiles of a tile odd and even in number, ragged last tiles
    (22, 56, 56, 64, 1, 8, 0, False), (29, 47, 49, 64, 1, 8, 1, True), (73, 30, 31, 64, 1, 8, 2, True), (242, 16, 17, 64, 1, 8, 1, False), (52, 33, 39, 64, 1, 8, 0, False),
    (64, 56, 56, 64, 1, 8, None, True), (33, 56, 55, 64, 1, 8, None, False),               # without one
    (9, 73, 77, 64, 1, 8, None, False), (8, 93, 101, 128, 1, 8, 1, False), (17, 56, 56, 192, 1, 8, None, True), (6, 112, 111, 64, 1, 4, 2, True),
    (20, 75, 63, 128, 2, 8, None, False), (200, 31, 29, 128, 2, 8, 0, False), (48, 61, 61, 192, 2, 8, None, True), (110, 45, 47, 256, 2, 8, 1, False),
    (90, 56, 55, 128, 2, 4, None, True), (30, 93, 95, 64, 2, 4, 2, True),
])
def test_whole_rows_at_the_sizes_that_reach_them(hawq, N, H, W, K, stride, bits, res, y4):
    """On both sides of the lines between this kernel and the others the same results; here the sizes past them."""
    test_whole_rows_64_channels(hawq, N, H, W, K, stride, bits, res, y4)


@pytest.mark.parametrize("N,H,W,K,stride,bits,res,y4", [
    (1024, 64, 1, 64, 1, 8, None, False), (300, 101, 2, 64, 1, 8, 0, False), (250, 67, 3, 64, 1, 8, 1, False),
    (500, 50, 1, 64, 2, 8, None, False), (200, 200, 2, 64, 2, 8, 0, False), (150, 91, 3, 128, 2, 8, None, True), (600, 177, 2, 64, 2, 4, None, True),
])
def test_outputs_one_to_three_pixels_wide(hawq, N, H, W, K, stride, bits, res, y4):
    """An output one pixel wide has no 32-bit reciprocal of its width: those layers run on the general kernels."""
    test_whole_rows_64_channels(hawq, N, H, W, K, stride, bits, res, y4)


@pytest.mark.parametrize("N,H,W,K,stride", [(9, 74, 73, 4160, 2), (8, 78, 80, 8320, 2), (9, 74, 73, 4096, 2)])
def test_many_output_channels(hawq, N, H, W, K, stride):
    """More than 64 groups of output channels leave the kernel too few workgroups along the pixels: the general kernels."""
    test_whole_rows_64_channels(hawq, N, H, W, K, stride, 8, None, False)
