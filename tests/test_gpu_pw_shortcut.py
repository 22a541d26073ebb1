"""GPU parity of the streaming 1x1 kernels, bit-exact: 128 input channels with a shortcut (ragged pixel groups and channel tiles, both
operand widths, every shortcut type, at the fewest pixels the kernel takes and beyond one round of its waves), and the walks of
the persistent kernels' waves over the XCDs."""
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
# workgroup's waves; the form with shared stages; the resident-weight 3x3, a number of tiles that is no multiple of 8.  All of them
# below the line of the eighths: their waves take turns.
@pytest.mark.parametrize("N,H,W,C,K,R,bits,res", [(1, 57, 144, 64, 64, 1, 8, False), (1, 57, 144, 64, 96, 1, 4, True), (1, 59, 141, 128, 96, 1, 8, False),
                                                  (1, 57, 144, 256, 64, 1, 4, False), (1, 57, 144, 256, 384, 1, 8, True), (11, 55, 55, 64, 64, 3, 8, True),
                                                  (13, 53, 51, 64, 64, 3, 4, False)])
def test_turns_with_uneven_shares(N, H, W, C, K, R, bits, res):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as hawq
    from gpu_util import run_conv_gpu, assert_same
    from test_gpu_conv import _scale_c
    case = _scale_c(wl.conv_case(seed=N + H + W + K, N=N, H=H, W=W, C=C, K=K, R=R, S=R, stride=1, pad=R // 2, bits=bits, with_residual=res), bits)
    x_dt, w_dt, hi = (hawq.U8, hawq.S8, 127) if bits == 8 else (hawq.U4, hawq.S4, 15)
    got, want = run_conv_gpu(case, x_dt, w_dt, x_dt, res_dt=x_dt, y_lo=0, y_hi=hi, x_hi=127 if bits == 8 else 0)
    assert_same(got, want, str((N, H, W, C, K, R, bits, res)))


def _sequences(slots, n_ct, groups, even):
    """How many walks over the pixel groups a launch makes (stream_sequences of csrc/xcd_walk.h)."""
    n = max(1, min(slots // n_ct, groups))
    if slots // n_ct >= groups:
        return -(-groups // 8) * 8 if even and slots // n_ct >= -(-groups // 8) * 8 else groups
    return n // 8 * 8 if even and 33 * (n // 8 * 8) >= 32 * n else n


# a number of sequences that is no multiple of 8, so that they are not dealt evenly over the XCDs: (pixels, C, K, bits, shortcut, the
# launch's waves, pixels of a group)
@pytest.mark.parametrize("M,C,K,bits,res,slots,px", [(8777, 64, 1184, 8, False, 4096, 32), (13801, 128, 624, 8, False, 2048, 64), (9001, 128, 832, 4, False, 2048, 64),
                                                     (8713, 128, 832, 8, True, 2048, 32), (8713, 128, 1264, 4, True, 3072, 32),
                                                     (8207, 256, 1408, 8, True, 2048, 32), (9747, 256, 640, 8, False, 3072, 32)])
def test_sequences_not_dealt_evenly(M, C, K, bits, res, slots, px):
    assert _sequences(slots, (K + 31) // 32, -(-M // px), C < 256) % 8 != 0
    test_turns_with_uneven_shares(1, 1, M, C, K, 1, bits, res)


@pytest.mark.parametrize("N,H,C,K,Cs,ss,slots", [(2, 68, 64, 896, 64, 1, 4096), (3, 60, 128, 384, 256, 2, 2048)])
def test_two_convolutions_with_sequences_not_dealt_evenly(N, H, C, K, Cs, ss, slots):
    import paper_2011_10680_amd as hawq
    from gpu_util import assert_same
    from test_gpu_dual import _case, _run
    assert _sequences(slots, K // 32, -(-N * H * H // 32), False) % 8 != 0
    got, want = _run(hawq, _case(N + H + K, N, H, C, K, 1, Cs, ss), hawq.U8, 1, 0, 127)
    assert_same(got, want, str((N, H, C, K, Cs, ss)))


def _line():
    """Output pixels from which the persistent kernels walk an XCD's own eighth (xcd_eighths of csrc/xcd_walk.h)."""
    import pathlib
    import re
    import paper_2011_10680_amd as hawq
    return int(re.search(r"bool xcd_eighths\(int64_t pixels\) { return pixels >= (\d+); }",
                         (pathlib.Path(hawq.__file__).parent / "csrc" / "xcd_walk.h").read_text())[1])


# eighths of unequal size: 397 and 403 tiles of 128 pixels, 1587 and 1611 groups of 32 (no multiple of 8), ragged at the end; the 3x3 with
# resident weights, the kernel with stages of a wave's own, the ones with shared stages
@pytest.mark.parametrize("N,H,W,C,K,R,bits,res", [
    (13, 63, 62, 64, 64, 3, 8, False), (13, 63, 62, 64, 64, 3, 8, True), (13, 63, 62, 64, 64, 3, 4, False), (13, 63, 62, 64, 64, 3, 4, True),
    (13, 63, 62, 64, 64, 1, 8, False), (13, 63, 62, 64, 96, 1, 4, False), (13, 63, 62, 64, 256, 1, 4, True), (4, 113, 114, 128, 128, 1, 8, True),
    (4, 113, 114, 256, 384, 1, 8, False), (4, 113, 114, 256, 128, 1, 4, True),
])
def test_eighths_of_unequal_size(N, H, W, C, K, R, bits, res):
    assert N * H * W >= _line() and -(-N * H * W // 128) % 8 and -(-N * H * W // 32) % 8
    test_turns_with_uneven_shares(N, H, W, C, K, R, bits, res)


@pytest.mark.parametrize("N,H,C,K,Cs,ss", [(13, 63, 64, 256, 64, 1), (13, 63, 64, 256, 64, 2), (13, 63, 128, 512, 256, 2)])
def test_two_convolutions_in_eighths(N, H, C, K, Cs, ss):
    import paper_2011_10680_amd as hawq
    from gpu_util import assert_same
    from test_gpu_dual import _case, _run
    assert N * H * H >= _line() and -(-N * H * H // 32) % 8
    got, want = _run(hawq, _case(N + H + K, N, H, C, K, 1, Cs, ss), hawq.U8, 1, 0, 127)
    assert_same(got, want, str((N, H, C, K, Cs, ss)))
