"""GPU parity: ResNet50's 64-channel bottleneck blocks as one launch each, vs the CPU oracle, bit-exact, at the sizes where a tile of
14 x 8 pixels, the walk over the tiles or a second workgroup on a compute unit can go wrong, and in every storage form."""
import numpy as np
import pytest

from oracle import resnet as onet
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hawq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2011_10680_amd as h
    h.load_library()
    return h


def _bits(four):
    """All 8-bit but the named groups of stage 1 (block, convolution) and whatever follows it."""
    b = {g: 8 for g in wl.resnet_group_names(50)}
    if four == "all":
        return {g: (8 if g in ("conv1", "fc") else 4) for g in b}
    for g in four:
        assert g in b, sorted(b)[:12]
        b[g] = 4
    return b


def _forward(hawq, net, x, mode=0):
    """(logits, how many of stage 1's steps do work)"""
    import torch
    N = x.shape[0]
    try:
        hawq.hawq_tune_set_fusion(mode)
        hn = hawq.HawqNet(50, net["layers"], net["pool_b"], net["pool_c"], image_hw=net["image_hw"])
    finally:
        hawq.hawq_tune_set_fusion(0)
    ws = torch.full((hn.workspace_bytes(N),), 0x7B, dtype=torch.uint8, device="cuda")
    logits = torch.zeros((N, 1000), dtype=torch.int32, device="cuda")
    xd = torch.from_numpy(x).cuda()
    for _ in range(2):
        hn.hawq_forward_resnet(xd, N, logits, ws)
    torch.cuda.synchronize()
    working = sum(hn.step_cost(N, s)[0] > 0 for s in range(hn.num_steps()) if hn.step_output(N, s)["name"].startswith("layer1"))
    out = logits.cpu().numpy()
    hn.close()
    return out, working


# map side = image side / 4: 8 (one tile, 8 of 14 columns), 16 (2 columns in the second tile), 25 (11 columns, one row), 56 (exact);
# tiles: up to 256 (one workgroup a unit), 280 (some units two), 672 (a walk of more than one tile); 33 x 33 at 80 images: 1200
@pytest.mark.parametrize("hw,N,four,int32_sc", [
    (32, 1, (), True), (64, 3, (), False), (100, 2, "all", True), (100, 3, "all", False), (224, 10, (), True), (224, 24, (), False),
    (132, 80, "all", False), (224, 1, ("layer1.1.in",), True), (64, 5, ("layer1.0.c2", "layer1.2.in", "layer1.2.c3"), False),
    (100, 4, ("layer2.0.in", "layer1.1.c3"), False), (64, 260, (), True),
    (100, 3, ("layer1.0.c3",), True), (100, 3, ("layer1.0.c2", "layer1.0.c3"), False)])
def test_blocks_as_one_launch(hawq, hw, N, four, int32_sc):
    net = wl.make_resnet(50, seed=900 + hw + N, bits=_bits(four), image_hw=hw, int32_shortcut=int32_sc)
    x = wl.make_image_batch(901 + N, N, image_hw=hw)
    got, working = _forward(hawq, net, x)
    assert np.array_equal(got, onet.forward(net, x))
    assert working == 3, working


@pytest.mark.parametrize("arch", [18, 50])
def test_last_convolutions_of_four_bits_with_an_int32_shortcut(hawq, arch):
    """A transition layer of 8 bits and a last convolution of 4, both branches INT32: one launch, no raw accumulators in memory."""
    import torch
    last = "c3" if arch == 50 else "c2"
    bits = {g: (4 if g.endswith(".0." + last) else 8) for g in wl.resnet_group_names(arch)}
    assert sum(b == 4 for b in bits.values()) == 4
    net = wl.make_resnet(arch, seed=83 + arch, bits=bits, image_hw=64, int32_shortcut=True)
    x = wl.make_image_batch(84, 3, image_hw=64)
    hn = hawq.HawqNet(arch, net["layers"], net["pool_b"], net["pool_c"], image_hw=64)
    ws = torch.full((hn.workspace_bytes(3),), 0x7B, dtype=torch.uint8, device="cuda")
    logits = torch.zeros((3, 1000), dtype=torch.int32, device="cuda")
    hn.hawq_forward_resnet(torch.from_numpy(x).cuda(), 3, logits, ws)
    torch.cuda.synchronize()
    names = [hn.step_output(3, s)["name"] for s in range(hn.num_steps())]
    got = logits.cpu().numpy()
    hn.close()
    assert not [n for n in names if n.endswith(".acc")], names
    assert np.array_equal(got, onet.forward(net, x))


@pytest.mark.parametrize("int32_sc", [True, False])
@pytest.mark.parametrize("mode", [0, -1])
def test_steps_that_leave_no_output_say_so(hawq, mode, int32_sc):
    """A convolution whose work a later step's launch does reports an empty output, every other one (conv1, whose pool is computed with it,
    and the classifier aside) where it is."""
    net = wl.make_resnet(50, seed=85, image_hw=64, int32_shortcut=int32_sc)
    try:
        hawq.hawq_tune_set_fusion(mode)
        hn = hawq.HawqNet(50, net["layers"], net["pool_b"], net["pool_c"], image_hw=64)
    finally:
        hawq.hawq_tune_set_fusion(0)
    steps = [(hn.step_output(3, s), hn.step_cost(3, s)[0]) for s in range(hn.num_steps())]
    hn.close()
    empty = [o["name"] for o, _ in steps if o["bytes"] == 0]
    inner = ["layer1.%d.c%d" % (b, c) for b in range(3) for c in (1, 2)] if mode == 0 else []
    ds = [] if int32_sc else ["layer%d.0.ds" % l for l in (1, 2, 3, 4)]
    assert sorted(empty) == sorted(["conv1", "fc"] + inner + ds)
    assert all(o["bytes"] == 0 for o, macs in steps if macs == 0 and o["name"] not in ("pool", "avgpool"))


def test_blocks_with_large_shortcut_multipliers(hawq):
    """Shortcut multipliers of 16 bits and more: the integer form of that term, still as one launch."""
    net = wl.make_resnet(50, seed=79, image_hw=64)
    for name in ("layer1.1.c3", "layer1.2.c3"):
        l = next(l for l in net["layers"] if l["name"] == name)
        sel = np.arange(256) % 9 == 4
        l["res_b"] = np.where(sel, l["res_b"].astype(np.int64) << 3, l["res_b"]).astype(np.int32)
        l["res_c"] = np.where(sel, l["res_c"].astype(np.int32) + 3, l["res_c"]).astype(np.uint8)
        assert l["res_b"].max() >= 65536
    x = wl.make_image_batch(80, 3, image_hw=64)
    got, working = _forward(hawq, net, x)
    assert np.array_equal(got, onet.forward(net, x)) and working == 3, working


@pytest.mark.parametrize("shifts,multipliers", [
    (range(2, 9), lambda g, c: np.minimum(g.integers(0, 6, 256) << np.maximum(c - 4, 0), 65535)),          # the smallest shifts: sums of whole, half and quarter steps
    (range(14, 18), lambda g, c: np.where(g.random(256) < 0.5, 1 << np.minimum(c - 1, 15), 65535 - g.integers(0, 3, 256))),   # halves; the largest multipliers
    (range(22, 28), lambda g, c: g.choice([1 << 15, 65535, 65534, 0], 256)),                              # steps of a 128th of one and less
    (range(24, 31), lambda g, c: g.choice([1 << 15, 65535, 65534, 0], 256))])                             # the largest shifts: nothing left
def test_blocks_with_shortcut_multipliers_at_the_ends_of_the_float_form(hawq, shifts, multipliers):
    """Shortcuts in floating point where a product meets a half, and at either end of its multipliers and shifts."""
    net = wl.make_resnet(50, seed=87, image_hw=64)
    g = np.random.default_rng(shifts[0])
    for name in ("layer1.1.c3", "layer1.2.c3"):
        l = next(l for l in net["layers"] if l["name"] == name)
        c = g.choice(np.array(shifts), 256)
        c[:len(shifts)] = shifts
        l["res_c"], l["res_b"] = c.astype(np.uint8), multipliers(g, c).astype(np.int32)
        # (one launch: multipliers raised to the largest shift stay below 2^22)
        assert l["res_b"].max() < 65536 and (l["res_b"].astype(np.int64) << (c.max() - c)).max() < 1 << 22
    x = wl.make_image_batch(88, 3, image_hw=64)
    got, working = _forward(hawq, net, x)
    assert np.array_equal(got, onet.forward(net, x)) and working == 3, working


@pytest.mark.parametrize("int32_sc", [True, False])
@pytest.mark.parametrize("what", ["wide", "bias"])
def test_blocks_beyond_the_narrow_evaluation(hawq, what, int32_sc):
    """A multiplier beyond the narrow evaluation's range, or a bias with which an accumulator may pass 32 bits: that block keeps its
    own launches, the others do not; same logits as the plan without fusion."""
    net = wl.make_resnet(50, seed=77, image_hw=64, int32_shortcut=int32_sc)
    l = next(l for l in net["layers"] if l["name"] == "layer1.1.c2")
    if what == "wide":
        l["b"] = np.where(np.arange(64) == 5, l["b"].astype(np.int64) << 15, l["b"]).astype(np.int32)
        l["c"] = np.where(np.arange(64) == 5, l["c"].astype(np.int32) + 15, l["c"]).astype(np.uint8)
    else:
        l["bias"] = np.where(np.arange(64) == 5, 2 ** 31 - 1000, l["bias"]).astype(np.int32)
    x = wl.make_image_batch(78, 2, image_hw=64)
    got, working = _forward(hawq, net, x)
    plain, separate = _forward(hawq, net, x, -1)
    assert np.array_equal(got, plain) and working == 5 and separate >= 9, (working, separate)
    if what == "wide":
        assert np.array_equal(got, onet.forward(net, x))


def test_measured_latencies_of_a_joined_block(hawq):
    """A block's launch has one time.  In the table of the bit selection the widths that the launch does not see (its second and third
    convolution, and the transition block's first, whose input is bytes at both) cost the same, and no time is lost."""
    import torch
    from paper_2011_10680_amd import bitselect as bs
    N, hw = 2, 64
    nets, total = {}, {}
    for b in (4, 8):
        net = wl.make_resnet(50, seed=5, bits=_bits("all" if b == 4 else ()), image_hw=hw)
        nets[b] = hawq.HawqNet(50, net["layers"], net["pool_b"], net["pool_c"], image_hw=hw)
        timed, total[b] = nets[b].hawq_forward_resnet_timed, []
        nets[b].hawq_forward_resnet_timed = lambda *a, timed=timed, b=b: total[b].append(timed(*a)) or total[b][-1]
    names, Q = bs.measure_group_latencies(nets, N, torch.from_numpy(wl.make_image_batch(6, N, image_hw=hw)).cuda(), repeats=2)
    cost_names, _, _ = bs.layer_costs(50, image_hw=hw, choices=(8,))
    for hn in nets.values():
        hn.close()
    assert names == cost_names and np.all(Q > 0)
    for name in ("layer1.0.c1", "layer1.0.c2", "layer1.0.c3", "layer1.1.c2", "layer1.1.c3", "layer1.2.c2", "layer1.2.c3"):
        q = Q[names.index(name)]
        assert np.isclose(q[0], q[1], rtol=1e-12), (name, q)
    assert np.allclose(Q.sum(axis=0), [np.median(np.array(total[b]), axis=0).sum() for b in (4, 8)], rtol=1e-12)
