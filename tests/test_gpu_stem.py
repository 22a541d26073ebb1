"""GPU parity: the first convolution with its max pool as the networks run it, vs the CPU oracle, bit-exact, at image sizes that leave
every remainder of the 8 x 8 pooled tiles, at batches of one tile a workgroup and of several, and in both output forms."""
import numpy as np
import pytest

from oracle import resnet as onet
import workloads as wl

pytestmark = pytest.mark.gpu


# pooled side = image side / 4: 8 (one tile), 9 (one pixel in the second), 15, 17, 25, 56, 57; 25 x 25 at 40 images: 640 tiles
@pytest.mark.parametrize("hw,N,four,wide", [(32, 1, False, False), (36, 3, False, True), (60, 2, True, False), (68, 2, False, False),
                                            (100, 40, False, False), (100, 3, True, True), (224, 12, True, False), (228, 2, False, True)])
def test_stem_with_pool(hw, N, four, wide):
    import torch
    import paper_2011_10680_amd as hawq
    bits = {g: (8 if g in ("conv1", "fc") or not four else 4) for g in wl.resnet_group_names(18)}
    net = wl.make_resnet(18, seed=500 + hw, bits=bits, image_hw=hw)
    if wide:          # numerators beyond the narrow evaluation's range: same values, the 64-bit form
        l = net["layers"][0]
        l["b"] = np.where(np.arange(64) % 7 == 3, l["b"].astype(np.int64) << 15, l["b"]).astype(np.int32)
        l["c"] = np.where(np.arange(64) % 7 == 3, l["c"].astype(np.int32) + 15, l["c"]).astype(np.uint8)
    x = wl.make_image_batch(501 + N, N, image_hw=hw)
    x[0, 0], x[0, -1], x[0, :, 0], x[0, :, -1] = 255, 0, 255, 0          # (the offset's extremes along the padding)
    hn = hawq.HawqNet(18, net["layers"], net["pool_b"], net["pool_c"], image_hw=hw)
    ws = torch.full((hn.workspace_bytes(N),), 0x7B, dtype=torch.uint8, device="cuda")
    logits = torch.zeros((N, 1000), dtype=torch.int32, device="cuda")
    hn.hawq_forward_resnet(torch.from_numpy(x).cuda(), N, logits, ws)
    torch.cuda.synchronize()
    got = logits.cpu().numpy()
    hn.close()
    assert np.array_equal(got, onet.forward(net, x))
