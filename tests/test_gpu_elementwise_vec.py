"""GPU parity of the vector forms of the memory-bound operators at the edges of their grids, bit-exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hawq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as h
    h.load_library()
    return h


def _draw(g, shape, dt):
    lo, hi, t = {oracle.S32: (-(1 << 18), 1 << 18, np.int32), oracle.U8: (0, 256, np.uint8), oracle.S8: (-128, 128, np.int8)}[dt]
    return g.integers(lo, hi, size=shape).astype(t)


# one unit; fewer units than a workgroup; K / 4 odd (the grid is a multiple of it); several rounds of four and a remainder;
# more channel groups than the largest grid has workgroups (element-wise form)
@pytest.mark.parametrize("P,K", [(1, 4), (37, 12), (101, 4 * 77), (5003, 256), (70001, 64), (3, 4 * 4099)])
@pytest.mark.parametrize("m_dt,r_dt,y_dt", [(oracle.S32, oracle.U8, oracle.U8), (oracle.S8, oracle.S32, oracle.S32), (oracle.U8, oracle.S8, oracle.S8)])
def test_residual_add_vector_form(hawq, P, K, m_dt, r_dt, y_dt):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(P + K)
    m, r = _draw(g, (P, K), m_dt), _draw(g, (P, K), r_dt)
    dn = lambda dt: (g.integers(1 << 14, 1 << 15, size=K).astype(np.int32), (g.integers(0, 2, size=K) + (27 if dt == oracle.S32 else 15)).astype(np.uint8))
    (mb, mc), (rb, rc) = dn(m_dt), dn(r_dt)
    lo, hi = {oracle.U8: (0, 127), oracle.S8: (-128, 127), oracle.S32: (-1000, 1000)}[y_dt]
    y = torch.full((P, K), 0x5A, dtype={oracle.U8: torch.uint8, oracle.S8: torch.int8, oracle.S32: torch.int32}[y_dt], device="cuda")
    hawq.hawq_residual_add_dyadic(P, K, m_dt, r_dt, y_dt, to_dev(m), to_dev(mb), to_dev(mc), to_dev(r), to_dev(rb), to_dev(rc), 0, lo, hi, y)
    torch.cuda.synchronize()
    want = oracle.residual_add_dyadic(m, mb, mc, r, rb, rc, n_pixels=P, K=K, m_dt=m_dt, r_dt=r_dt, y_dt=y_dt, relu=0, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy(), want.reshape(P, K))


# both sides of the streaming form's line (400000 or, with an INT32 operand, 900000 groups of four), a channel group count that does
# not divide the grid, in narrow parameters, with one channel outside the INT32 form's range (c > 32) and outside the 8-bit form's (b >= 2^22)
@pytest.mark.parametrize("P,K,m_dt,r_dt,y_dt", [(56249, 64, oracle.S32, oracle.U8, oracle.U8), (56251, 64, oracle.S32, oracle.U8, oracle.U8),
                                                (11689, 4 * 77, oracle.S32, oracle.S32, oracle.S32), (3127, 512, oracle.U8, oracle.S8, oracle.S8),
                                                (5201, 4 * 77, oracle.S8, oracle.U8, oracle.U8),
                                                # grids of 750 workgroups (the next multiple, 775, above 768) and of 771 (the one below is 514)
                                                (36011, 100, oracle.S32, oracle.U8, oracle.U8), (3503, 1028, oracle.S32, oracle.S8, oracle.U8)])
@pytest.mark.parametrize("wide", [None, "c", "b"])
def test_residual_add_streaming_form(hawq, P, K, m_dt, r_dt, y_dt, wide):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(P + K)
    m, r = _draw(g, (P, K), m_dt), _draw(g, (P, K), r_dt)
    dn = lambda dt: (g.integers(1 << 14, 1 << 15, size=K).astype(np.int32), (g.integers(0, 2, size=K) + (27 if dt == oracle.S32 else 15)).astype(np.uint8))
    (mb, mc), (rb, rc) = dn(m_dt), dn(r_dt)
    if wide == "c":
        mb[K // 2], mc[K // 2] = (1 << 31) - 1, 43
    if wide == "b":
        rb[5], rc[5] = 3 << 22, 24
    lo, hi = {oracle.U8: (0, 127), oracle.S8: (-128, 127), oracle.S32: (-1000, 1000)}[y_dt]
    y = torch.full((P, K), 0x5A, dtype={oracle.U8: torch.uint8, oracle.S8: torch.int8, oracle.S32: torch.int32}[y_dt], device="cuda")
    hawq.hawq_residual_add_dyadic(P, K, m_dt, r_dt, y_dt, to_dev(m), to_dev(mb), to_dev(mc), to_dev(r), to_dev(rb), to_dev(rc), 0, lo, hi, y)
    torch.cuda.synchronize()
    want = oracle.residual_add_dyadic(m, mb, mc, r, rb, rc, n_pixels=P, K=K, m_dt=m_dt, r_dt=r_dt, y_dt=y_dt, relu=0, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy(), want.reshape(P, K))


# narrow parameters, and one channel with c > 32; fewer units than threads, several rounds of four and a remainder
@pytest.mark.parametrize("P", [3, 30011])
def test_concat_wide_parameters(hawq, P):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(P)
    host, dev = [], []
    for K, dt in ((64, oracle.S32), (12, oracle.U8)):
        q = _draw(g, (P, K), dt)
        b = g.integers(1 << 14, 1 << 15, size=K).astype(np.int32)
        c = np.full(K, 27 if dt == oracle.S32 else 15, dtype=np.uint8)
        b[7], c[7] = (1 << 30) + 12345, 44 if dt == oracle.S32 else 31
        host.append((q, dt, b, c))
        dev.append((to_dev(q), dt, to_dev(b), to_dev(c)))
    y = torch.full((P, 76), 0x5A, dtype=torch.uint8, device="cuda")
    hawq.hawq_concat_dyadic(P, dev, oracle.U8, 0, 127, y)
    torch.cuda.synchronize()
    want = oracle.concat_dyadic(host, n_pixels=P, y_dt=oracle.U8, y_lo=0, y_hi=127)
    assert_same(y.cpu().numpy(), np.asarray(want).reshape(tuple(y.shape)))


# INT32 operands past the caches: from 128 MB in all on; one group of four below and above, results of either width
@pytest.mark.parametrize("P,K,m_dt,r_dt,y_dt", [(41666, 512, oracle.S32, oracle.U8, oracle.U8), (41667, 512, oracle.S8, oracle.S32, oracle.U8),
                                                (26044, 4 * 103, oracle.S32, oracle.S32, oracle.S32)])
def test_residual_add_past_the_caches(hawq, P, K, m_dt, r_dt, y_dt):
    test_residual_add_streaming_form(hawq, P, K, m_dt, r_dt, y_dt, "c")


# the form of large tensors, from 2^22 groups of four on: narrow parameters, and waves that hold a channel outside their range beside
# others; an even and an odd number of pixels left to a thread
@pytest.mark.parametrize("P,y_dt", [(43701, oracle.U8), (43700, oracle.U4), (54613, oracle.S32)])
@pytest.mark.parametrize("wide", [False, True])
def test_concat_large_form(hawq, P, y_dt, wide):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(P)
    host, dev = [], []
    for K, dt in ((228, oracle.S32), (100, oracle.U8), (56, oracle.S8)):
        q = _draw(g, (P, K), dt)
        b = g.integers(1 << 14, 1 << 15, size=K).astype(np.int32)
        c = np.full(K, 27 if dt == oracle.S32 else 15, dtype=np.uint8)
        if wide:
            b[K // 2], c[K // 2] = (1 << 30) + 12345, 44 if dt == oracle.S32 else 31
        host.append((q, dt, b, c))
        dev.append((to_dev(q), dt, to_dev(b), to_dev(c)))
    lo, hi = {oracle.U8: (0, 127), oracle.U4: (0, 15), oracle.S32: (-1000, 1000)}[y_dt]
    assert P * 96 >= 1 << 22
    y = torch.full((P, 192 if y_dt == oracle.U4 else 384), 0x5A, dtype=torch.int32 if y_dt == oracle.S32 else torch.uint8, device="cuda")
    hawq.hawq_concat_dyadic(P, dev, y_dt, lo, hi, y)
    torch.cuda.synchronize()
    want = oracle.concat_dyadic(host, n_pixels=P, y_dt=y_dt, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy(), np.asarray(want).reshape(tuple(y.shape)))


@pytest.mark.parametrize("P,spec,y_dt", [(1, [(4, oracle.S32)], oracle.U8), (777, [(64, oracle.S32), (12, oracle.U8), (4, oracle.S8)], oracle.U8),
                                         (9000, [(64, oracle.S32), (64, oracle.S32), (96, oracle.S32), (288, oracle.S32)], oracle.U8),
                                         (50, [(4, oracle.S32)] * 8, oracle.S32), (50, [(8, oracle.U8)] * 9, oracle.U8),
                                         (301, [(20, oracle.S32), (8, oracle.U8)], oracle.U4)])
def test_concat_in_one_launch(hawq, P, spec, y_dt):
    import torch
    from gpu_util import to_dev, assert_same
    g = np.random.default_rng(P)
    lo, hi = {oracle.U8: (0, 127), oracle.U4: (0, 15), oracle.S32: (-5000, 5000)}[y_dt]
    host, dev = [], []
    for K, dt in spec:
        q = _draw(g, (P, K), dt)
        b = g.integers(1 << 14, 1 << 15, size=K).astype(np.int32)
        c = (g.integers(0, 2, size=K) + (27 if dt == oracle.S32 else 15) + (3 if hi == 15 else 0)).astype(np.uint8)
        host.append((q, dt, b, c))
        dev.append((to_dev(q), dt, to_dev(b), to_dev(c)))
    Kt = sum(K for K, _ in spec)
    y = torch.full((P, Kt // 2 if y_dt == oracle.U4 else Kt), 0x5A, dtype=torch.int32 if y_dt == oracle.S32 else torch.uint8, device="cuda")
    hawq.hawq_concat_dyadic(P, dev, y_dt, lo, hi, y)
    torch.cuda.synchronize()
    want = oracle.concat_dyadic(host, n_pixels=P, y_dt=y_dt, y_lo=lo, y_hi=hi)
    assert_same(y.cpu().numpy(), np.asarray(want).reshape(tuple(y.shape)))


@pytest.mark.parametrize("N,H,W,C", [(1, 1, 1, 4), (4, 17, 17, 64), (9, 17, 18, 256), (30, 35, 33, 64)])
def test_pool3x3_patch_sizes(hawq, N, H, W, C):
    """Single outputs, 2x2 and 4x4 patches per thread, with ragged borders."""
    import torch
    from gpu_util import to_dev, assert_same
    x = np.random.default_rng(C + H).integers(0, 1 << 20, size=(N, H, W, C)).astype(np.int32)
    y = torch.full((N, H, W, C), 0x5A, dtype=torch.int32, device="cuda")
    hawq.hawq_pool2d_sum_int(N, H, W, C, 3, 3, 1, 1, 1, 1, hawq.S32, hawq.S32, to_dev(x), None, None, 0, 0, y)
    torch.cuda.synchronize()
    want = oracle.pool2d_sum_int(x, None, None, N=N, H=H, W=W, C=C, R=3, S=3, stride=1, pad=1, x_dt=oracle.S32, y_dt=oracle.S32)
    assert_same(y.cpu().numpy(), want)


@pytest.mark.parametrize("N,H,W,C", [(4, 35, 34, 768), (3, 29, 28, 1024), (4, 37, 38, 640)])
def test_pool3x3_patch_sizes_many_channels(hawq, N, H, W, C):
    test_pool3x3_patch_sizes(hawq, N, H, W, C)


@pytest.mark.parametrize("P", [4095, 4097])
@pytest.mark.parametrize("y_dt", [oracle.U8, oracle.U4])
def test_one_branch_on_both_sides_of_its_line(hawq, P, y_dt):
    """2^19 groups of four channels: one group per thread below, the walking form from there on."""
    test_concat_in_one_launch(hawq, P, [(512, oracle.S32)], y_dt)
