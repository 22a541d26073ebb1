"""The native marshalling of the per-layer entry points against the ctypes path, on the host: every call here is refused by the
library's argument checks before a launch, and must be refused in the same way, with the same values seen, by both."""
import ctypes

import numpy as np
import pytest


@pytest.fixture(scope="module")
def both():
    """call(name, *args): the outcome through the native path and through ctypes."""
    import torch
    import paper_2011_10680_amd as hawq
    import paper_2011_10680_amd.binding as B
    from paper_2011_10680_amd import build
    if build.is_stale():
        build.build()
    F = pytest.importorskip("paper_2011_10680_amd._fastcall", reason="the optional native module is not built")
    lib = hawq.load_library()
    names = ("conv2d_int", "conv2d_dual_int", "gemm_int", "residual_add_dyadic", "avgpool_int", "maxpool_int", "pool2d_sum_int", "concat_dyadic")
    addresses = tuple(ctypes.cast(getattr(lib, "hawq_" + n), ctypes.c_void_p).value for n in names)
    assert F.setup(addresses, torch.Tensor, torch.nn.Parameter, hawq.ConvDesc, lambda: 0, lambda d: 0)

    def outcome(f, args):
        try:
            return f(*args, stream=0)
        except hawq.HawqError as e:
            return e.status
        except Exception as e:
            return type(e)

    def call(name, *args):
        f, was = getattr(hawq, name), B._fast
        got = []
        for B._fast in (F, None):
            got.append(outcome(f, args))
        B._fast = was
        return got
    return call


def test_every_entry_point_is_refused_alike(both):
    import torch
    import paper_2011_10680_amd as hawq
    x = torch.zeros(64, dtype=torch.uint8)
    p = torch.nn.Parameter(torch.zeros(64), requires_grad=False)
    d = lambda **kw: hawq.ConvDesc(**dict(dict(N=1, H=8, W=8, C=64, K=64, R=3, S=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, x_dtype=0, w_dtype=1, y_hi=127), **kw))

    class Sub(torch.Tensor):
        pass
    sub = x.as_subclass(Sub)
    cases = [
        (2, "hawq_conv2d_int", d(H=0), x, x, x, x, x, None, None, None, x),
        (2, "hawq_conv2d_int", d(H=0), x, p, x, x, x, None, None, None, sub),
        (1, "hawq_conv2d_int", d(), x, x, x, x, x, x, None, None, x),
        (1, "hawq_conv2d_int", d(), None, x, x, x, x, None, None, None, x),
        (4, "hawq_conv2d_int", d(y_hi=300), x, x, x, x, x, None, None, None, x),
        (AttributeError, "hawq_conv2d_int", d(), 5, x, x, x, x, None, None, None, x),
        (ctypes.ArgumentError, "hawq_gemm_int", "1", 1, 64, 0, 1, 0, x, x, x, x, x, 1, 0, 127, x),
        (2, "hawq_conv2d_dual_int", d(R=11, S=11, pad_h=0, pad_w=0), x, x, x, x, x, d(R=1, S=1), x, x, x, x, x, x),
        (2, "hawq_gemm_int", 1, -1, 64, 0, 1, 0, x, x, x, x, x, 1, 0, 127, x),
        (2, "hawq_residual_add_dyadic", -1, 4, 0, 0, 0, x, x, x, x, x, x, 1, 0, 127, x),
        (3, "hawq_residual_add_dyadic", 1, 4, 0, 9, 0, x, x, x, x, x, x, 1, 0, 127, x),
        (2, "hawq_avgpool_int", 1, 0, 1, 64, 0, 0, x, x, x, 0, 127, x),
        (2, "hawq_maxpool_int", 1, 0, 1, 64, 0, 0, x, 0, 127, x),
        (2, "hawq_pool2d_sum_int", 1, 0, 4, 4, 3, 3, 1, 1, 1, 1, 4, 4, x, None, None, 0, 0, x),
        (1, "hawq_pool2d_sum_int", 1, 4, 4, 4, 3, 3, 1, 1, 1, 1, 4, 4, None, None, None, 0, 0, x),
        (2, "hawq_concat_dyadic", -1, [(x, 0, x, x)], 0, 0, 127, x),
        (3, "hawq_concat_dyadic", 1, [(x, 0, x, x), (x, 7, p, x)], 0, 0, 127, x),
        (4, "hawq_concat_dyadic", 1, [(x, 0, x, x)], 0, 5, 1, x),
        (4, "hawq_concat_dyadic", 1, [(x, 0, x, x)] * 40, 0, 5, 1, x),
        (4, "hawq_concat_dyadic", 1, tuple([(x, 0, x, x)]), 0, 5, 1, x),
    ]
    for want, name, *args in cases:
        native, plain = both(name, *args)
        assert native == plain == want, (name, native, plain, want)


def test_integers_of_other_types_and_out_of_range(both):
    """numpy integers and values past 32 / 64 bits: whatever ctypes makes of them."""
    import torch
    x = torch.zeros(64, dtype=torch.uint8)
    for v in (np.int32(-1), True, 1 << 32, (1 << 32) - 1, 1 << 70, -(1 << 70), 1.0):
        native, plain = both("hawq_avgpool_int", v, 0, 1, 64, 0, 0, x, x, x, 0, 127, x)
        assert native == plain, (v, native, plain)
