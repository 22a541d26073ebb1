"""GPU parity of the resident-pixel 1x1 kernel with a split reduction, bit-exact: every variant with ragged last tiles, strides,
shortcuts of every stored type, packed operands and outputs, parameters outside the narrow evaluation."""
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


# (N, H, W, C, K, stride, bits, shortcut dtype or None, 4-bit output)
@pytest.mark.parametrize("N,H,W,C,K,stride,bits,res,y4", [
    (3, 28, 29, 128, 512, 1, 8, 0, False), (9, 27, 27, 128, 128, 1, 4, 2, True),
    (5, 30, 30, 256, 64, 1, 8, None, False), (3, 13, 13, 256, 1024, 1, 8, 1, False), (7, 55, 57, 256, 128, 2, 8, None, True), (6, 14, 14, 256, 1024, 1, 4, 2, False),
    (7, 28, 27, 512, 64, 1, 8, None, False), (9, 7, 7, 512, 2048, 1, 8, 0, False), (11, 28, 28, 512, 256, 2, 8, None, False), (25, 7, 7, 512, 2048, 1, 4, 2, True),
    (5, 14, 13, 1024, 256, 1, 8, None, False), (31, 13, 14, 1024, 512, 2, 8, None, False), (17, 14, 14, 1024, 256, 1, 4, None, True),
    (5, 7, 7, 2048, 512, 1, 8, 1, False), (19, 7, 6, 2048, 512, 1, 8, None, True), (23, 7, 7, 2048, 512, 1, 4, None, True),
])
def test_pointwise_split_reduction(hawq, N, H, W, C, K, stride, bits, res, y4):
    import torch
    from gpu_util import to_dev, out_shape, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + C + K, N=N, H=H, W=W, C=C, K=K, R=1, S=1, stride=stride, pad=0, bits=bits,
                                 with_residual=res is not None, res_signed=res == 1), bits)
    if y4 and bits == 8:
        case["c"] = (case["c"] + 3).astype(np.uint8)
    if not y4 and bits == 4:
        case["c"] = (case["c"] - 3).astype(np.uint8)
    x_dt, w_dt = (hawq.U8, hawq.S8) if bits == 8 else (hawq.U4, hawq.S4)
    y_dt, hi = (hawq.U4, 15) if y4 else (hawq.U8, 127)
    P, Q = case["P"], case["Q"]
    d = hawq.ConvDesc(N=N, H=H, W=W, C=C, K=K, R=1, S=1, stride_h=stride, stride_w=stride, pad_h=0, pad_w=0, x_dtype=x_dt, w_dtype=w_dt,
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
        want = oracle.conv2d_int(case["x"], case["w"], case["bias"], b, c, N=N, H=H, W=W, C=C, K=K, R=1, S=1, stride=stride, pad=0, x_dt=x_dt,
                                 w_dt=w_dt, y_dt=y_dt, relu=1, y_lo=0, y_hi=hi, residual=case.get("residual") if res is not None else None,
                                 res_b=case.get("res_b"), res_c=case.get("res_c"), res_dt=res or 0)
        assert_same(y.cpu().numpy(), want, str((N, H, W, C, K, bits, wide)))
    v = oracle.unpack(want, oracle.U4) if y4 else want.astype(np.int32)
    assert 0.02 < (v > 0).mean() and (v == hi).mean() < 0.7
