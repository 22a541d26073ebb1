"""GPU parity of the resident-pixel 3x3 kernel with a split reduction (fragment-ordered weights, launches that do not fill the
chip), bit-exact: every channel count in both tile widths, ragged last tiles, tiles across image borders, images narrower
and wider than a tile, shortcuts, packed 4-bit operands and outputs, parameters outside the narrow evaluation."""
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


def _run(hawq, case, bits, y_dt, y_hi, res_dt=0):
    import torch
    from gpu_util import to_dev, out_shape
    N, H, W, C, K = (case[k] for k in ("N", "H", "W", "C", "K"))
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    d = hawq.ConvDesc(N=N, H=H, W=W, C=C, K=K, R=3, S=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, x_dtype=x_dt, w_dtype=w_dt, y_dtype=y_dt,
                      res_dtype=res_dt, relu=1, y_lo=0, y_hi=y_hi, x_hi=127 if bits == 8 else 0)
    w = to_dev(case["w"])
    wf = torch.empty(hawq.hawq_conv_fragment_weights_bytes(d), dtype=torch.uint8, device="cuda")
    hawq.hawq_conv_fragment_weights(d, w, wf)
    d.w_fragments = wf.data_ptr()
    y = torch.full(out_shape((N, H, W, K), y_dt), 0x5A, dtype=torch.uint8, device="cuda")
    res = case.get("residual")
    hawq.hawq_conv2d_int(d, to_dev(case["x"]), w, to_dev(case["bias"]), to_dev(case["b"]), to_dev(case["c"]), to_dev(res),
                         to_dev(case["res_b"]) if res is not None else None, to_dev(case["res_c"]) if res is not None else None, y)
    torch.cuda.synchronize()
    want = oracle.conv2d_int(case["x"], case["w"], case["bias"], case["b"], case["c"], N=N, H=H, W=W, C=C, K=K, R=3, S=3, stride=1, pad=1,
                             x_dt=x_dt, w_dt=w_dt, y_dt=y_dt, relu=1, y_lo=0, y_hi=y_hi, residual=res, res_b=case.get("res_b"),
                             res_c=case.get("res_c"), res_dt=res_dt)
    return y.cpu().numpy(), want


@pytest.mark.parametrize("N,H,W,C,K,bits,res,y4", [
    (6, 29, 31, 64, 64, 8, True, False), (5, 56, 56, 64, 128, 8, False, True), (9, 41, 23, 64, 64, 4, False, True),
    (2, 28, 28, 128, 128, 8, True, False), (9, 27, 29, 128, 128, 8, False, False), (3, 40, 41, 128, 192, 8, False, True), (9, 28, 28, 128, 128, 4, False, False),
    (3, 14, 14, 256, 256, 8, True, False), (11, 13, 15, 256, 256, 8, False, False), (2, 30, 29, 256, 256, 8, False, False), (17, 14, 14, 256, 256, 4, False, True),
    (5, 7, 7, 512, 512, 8, True, False), (31, 7, 7, 512, 512, 8, False, False), (3, 20, 20, 512, 512, 8, False, True), (17, 7, 7, 512, 512, 4, False, True),
    (70, 3, 2, 512, 512, 8, False, False),
])
def test_resident_pixels_split_reduction(hawq, N, H, W, C, K, bits, res, y4):
    from gpu_util import assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + W + C, N=N, H=H, W=W, C=C, K=K, R=3, S=3, stride=1, pad=1, bits=bits, with_residual=res,
                                 res_signed=res and K == 512), bits)
    if y4 and bits == 8:
        case["c"] = (case["c"] + 3).astype(np.uint8)
    if not y4 and bits == 4:
        case["c"] = (case["c"] - 3).astype(np.uint8)
    y_dt, hi = (hawq.U4, 15) if y4 else (hawq.U8, 127)
    got, want = _run(hawq, case, bits, y_dt, hi, hawq.S8 if (res and K == 512) else hawq.U8)
    assert_same(got, want, str((N, H, W, C, K, bits)))
    v = oracle.unpack(want, oracle.U4) if y4 else want.astype(np.int32)
    assert 0.02 < (v > 0).mean() and (v == hi).mean() < 0.6


def test_resident_pixels_split_reduction_wide_parameters(hawq):
    from gpu_util import assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=5, N=5, H=14, W=14, C=256, K=256, R=3, S=3, stride=1, pad=1, bits=8, with_residual=True), 8)
    got, want = _run(hawq, case, 8, hawq.U8, 127)
    assert_same(got, want)
    wide = dict(case, b=(case["b"].astype(np.int64) << 14).astype(np.int32), c=(case["c"].astype(np.int32) + 14).astype(np.uint8))
    got, want2 = _run(hawq, wide, 8, hawq.U8, 127)
    assert_same(got, want2)
    assert np.array_equal(want, want2)
