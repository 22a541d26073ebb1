"""GPU parity of the streaming 1x1 kernel with 128 input channels and a shortcut, bit-exact: ragged pixel groups and channel
tiles, both operand widths, every shortcut type, at the fewest pixels the kernel takes and beyond one round of its waves."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,K,bits,res", [
    (1, 64, 128, 512, 8, 0), (13, 28, 27, 512, 8, 1), (37, 28, 28, 528, 8, 0), (90, 28, 28, 512, 8, 0),
    (1, 64, 129, 512, 4, 2), (37, 28, 28, 512, 4, 2), (90, 29, 28, 528, 4, 2),
])
def test_128_channels_with_shortcut(N, H, W, K, bits, res):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as hawq
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + W + K, N=N, H=H, W=W, C=128, K=K, R=1, S=1, stride=1, pad=0, bits=bits,
                                 with_residual=True, res_signed=res == 1), bits)
    x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
    got, want = run_conv_gpu(case, x_dt, w_dt, x_dt, res_dt=res, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str((N, H, W, K, bits, res)))
    v = want.astype(np.int32) if bits == 8 else oracle.unpack(want, oracle.U4)
    assert 0.02 < (v > 0).mean() and len(np.unique(v)) > 5


@pytest.mark.parametrize("N,H,W,K,bits,res", [(1, 167, 98, 256, 4, 2), (1, 87, 147, 192, 8, 0), (1, 103, 129, 176, 8, 1), (1, 121, 137, 192, 4, 2)])
def test_128_channels_with_shortcut_in_one_round_of_tile_pairs(N, H, W, K, bits, res):
    test_128_channels_with_shortcut(N, H, W, K, bits, res)


# 8200-odd pixels: fewer groups than waves, so that some waves of an XCD have none; a channel count whose tiles do not divide a
# workgroup's waves; the form with shared stages; the resident-weight 3x3 with an uneven number of tiles per XCD
@pytest.mark.parametrize("N,H,W,C,K,R,bits,res", [(1, 57, 144, 64, 64, 1, 8, False), (1, 57, 144, 64, 96, 1, 4, True), (1, 59, 141, 128, 96, 1, 8, False),
                                                  (1, 57, 144, 256, 64, 1, 4, False), (1, 57, 144, 256, 384, 1, 8, True), (11, 55, 55, 64, 64, 3, 8, True),
                                                  (13, 53, 51, 64, 64, 3, 4, False)])
def test_walks_with_uneven_eighths(N, H, W, C, K, R, bits, res):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as hawq
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + W + K, N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, bits=bits, with_residual=res), bits)
    x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
    got, want = run_conv_gpu(case, x_dt, w_dt, x_dt, res_dt=x_dt, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str((N, H, W, C, K, R, bits, res)))
