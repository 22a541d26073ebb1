"""The native marshalling of the per-layer entry points on the host.  Against the ctypes path: calls that the library's argument checks
refuse before a launch must be refused in the same way by both.  By itself, over functions that record what they are called with: every
argument arrives in its place, and what the module leaves to the ctypes path reaches none of them."""
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
    yield call
    _restore()


def _restore():
    """The module as the binding uses it, where it does: with the device's own stream query."""
    import torch
    import paper_2011_10680_amd.binding as B
    if B._raw_stream is not None:
        B._use_fastcall(torch, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)


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


_NAMES = ("conv2d", "dual", "gemm", "residual_add", "avgpool", "maxpool", "pool2d_sum", "concat")
_ENTRIES = ("conv2d_int", "conv2d_dual_int", "gemm_int", "residual_add_dyadic", "avgpool_int", "maxpool_int", "pool2d_sum_int", "concat_dyadic")
_STREAM = 0x7A5C00


@pytest.fixture()
def recorder(both):
    """(module, calls): every entry point replaced by a function that records its arguments and returns 100 + its index."""
    import torch
    import paper_2011_10680_amd as hawq
    import paper_2011_10680_amd._fastcall as F
    lib, calls, kept = hawq.load_library(), [], []

    def record(i, types):
        def f(*args):
            # structures copied while the caller still holds them
            n = next((a for a, t in zip(args, types) if t is ctypes.c_int32), 0)
            seen = [(bytes(a[0]) if isinstance(a[0], hawq.ConvDesc) else [(b.q, b.dtype, b.K, b.b, b.c) for b in a[:n]])
                    if hasattr(a, "contents") else a for a in args]
            calls.append((i, seen))
            return 100 + i
        return ctypes.CFUNCTYPE(ctypes.c_int, *types)(f)

    for i, n in enumerate(_ENTRIES):
        kept.append(record(i, getattr(lib, "hawq_" + n).argtypes))
    addresses = tuple(ctypes.cast(f, ctypes.c_void_p).value for f in kept)
    assert F.setup(addresses, torch.Tensor, torch.nn.Parameter, hawq.ConvDesc, lambda: 3, lambda d: _STREAM + d)
    yield F, calls
    addresses = tuple(ctypes.cast(getattr(lib, "hawq_" + n), ctypes.c_void_p).value for n in _ENTRIES)
    assert F.setup(addresses, torch.Tensor, torch.nn.Parameter, hawq.ConvDesc, lambda: 0, lambda d: 0)
    _restore()
    kept.clear()


def _arguments(i):
    """Distinct arguments for entry point i and what the recorded call must show for them (its own stream: 77)."""
    import torch
    import paper_2011_10680_amd as hawq
    types = getattr(hawq.load_library(), "hawq_" + _ENTRIES[i]).argtypes
    store = torch.zeros(4096, dtype=torch.uint8)
    args, want = [], []
    for k, t in enumerate(types[:-1]):
        if t is ctypes.c_void_p:
            v = store[64 * k + 8:64 * k + 24]
            v = torch.nn.Parameter(v, requires_grad=False) if k % 3 == 0 else v
            args.append(v)
            want.append(v.data_ptr())
        elif t in (ctypes.c_int32, ctypes.c_int64):
            args.append((1 << 40) + k if t is ctypes.c_int64 else 1000 + k)
            want.append(args[-1])
        else:
            args.append(hawq.ConvDesc(N=k + 1, H=7, W=9, C=11 * k, y_hi=-k, x_hi=k))
            want.append(bytes(args[-1]))
    return args + [77], want + [77]


@pytest.mark.parametrize("i", range(7), ids=_NAMES[:7])
def test_every_argument_arrives_in_its_place(recorder, i):
    F, calls = recorder
    f = getattr(F, _NAMES[i])
    args, want = _arguments(i)
    assert f(*args) == 100 + i and calls == [(i, want)]
    calls.clear()
    assert f(*args[:-1], None) == 100 + i and calls == [(i, want[:-1] + [_STREAM + 3])]
    for k, v in enumerate(args[:-1]):
        if hasattr(v, "data_ptr"):
            calls.clear()
            assert f(*args[:k], None, *args[k + 1:]) == 100 + i and calls == [(i, want[:k] + [None] + want[k + 1:])]


@pytest.mark.parametrize("i", range(7), ids=_NAMES[:7])
def test_what_is_left_to_the_ctypes_path(recorder, i):
    import torch
    import paper_2011_10680_amd as hawq
    F, calls = recorder

    class SubTensor(torch.Tensor):
        pass

    class SubDesc(hawq.ConvDesc):
        pass
    f = getattr(F, _NAMES[i])
    args, _ = _arguments(i)
    for k, v in enumerate(args):
        if hasattr(v, "data_ptr"):
            others = [v.detach().as_subclass(SubTensor), 5, "x", np.zeros(4)]
        elif isinstance(v, int):
            others = [1.0, "1", np.int32(1)] + ([1 << 70, -(1 << 70)] if k + 1 < len(args) else [])
        else:
            others = [SubDesc(), None, 5]
        for o in others:
            assert f(*args[:k], o, *args[k + 1:]) is None, (k, o)
    assert f(*args[:-1]) is None and f(*args, 1) is None
    assert calls == []


def test_concatenation_branches(recorder):
    import torch
    F, calls = recorder
    store = torch.zeros(8192, dtype=torch.uint8)
    t = lambda k, n=16: store[64 * k:64 * k + n]
    branches = [(t(4 * j), j % 3, torch.nn.Parameter(t(4 * j + 1, 3 + j), requires_grad=False), t(4 * j + 2)) for j in range(32)]
    want = [(q.data_ptr(), dt, b.numel(), b.data_ptr(), c.data_ptr()) for q, dt, b, c in branches]
    for n in (0, 1, 2, 32):
        calls.clear()
        assert F.concat(1 << 40, branches[:n], 3, -5, 99, t(127), None) == 107
        (i, (pixels, count, seen, *rest)), = calls
        assert (i, pixels, count, seen if n else []) == (7, 1 << 40, n, want[:n]) and rest == [3, -5, 99, t(127).data_ptr(), _STREAM + 3]
    calls.clear()
    q, dt, b, c = branches[1]
    for wrong in (branches + branches[:1], tuple(branches), [(q, dt, b)], [[q, dt, b, c]], [(None, dt, b, c)], [(q, 1.0, b, c)], [(q, 1 << 70, b, c)], None):
        assert F.concat(1, wrong, 0, 0, 127, t(127), 0) is None, wrong
    assert calls == []
