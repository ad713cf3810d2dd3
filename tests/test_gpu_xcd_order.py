"""Kernels whose workgroups are ordered so that the k-th eighth of the pixels is XCD k's: units that do not divide by 8 or by the
workgroups, and both orders of the image-stationary kernel's workgroups, against the general kernel on the same operands and, for a few
images, the oracle."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# switches of the kernel, its name, image, channels in and out, window, batch
CASES = [
    # channels by channels (few units) and unit by unit (12 units of 14 x 14 are the line), with 4, 2 and 1 waves sharing K
    (dict(imgk=14), "conv3x3_imgk<256>", (14, 14), 256, 256, 3, 5), (dict(imgk=14), "conv3x3_imgk<256>", (14, 14), 256, 256, 3, 13),
    (dict(imgk=12), "conv3x3_imgk<256>", (14, 13), 256, 256, 3, 43), (dict(imgk=11), "conv3x3_imgk<256>", (13, 14), 256, 256, 3, 70),
    (dict(imgk=12), "conv3x3_imgk<512>", (7, 7), 512, 512, 3, 201), (dict(imgk=12), "conv3x3_imgk<128>", (28, 28), 128, 128, 3, 9),
    # persistent kernels: fewer units than workgroups, more, none a multiple of 8
    (dict(conv_img=2, conv_img_min=1, imgk=0), "conv3x3_img<256x256>", (14, 14), 256, 256, 3, 3),
    (dict(conv_img=2, conv_img_min=1, imgk=0), "conv3x3_img<256x256>", (9, 14), 256, 256, 3, 267),
    (dict(conv_img=2, conv_img_min=1, imgk=0), "conv3x3_img<128x128>", (30, 28), 128, 128, 3, 133),
    (dict(conv_ws_min=1, imgk=0, conv_img=0), "conv3x3_ws<64x64>", (20, 21), 64, 64, 3, 13), (dict(conv_ws_min=1, imgk=0, conv_img=0), "conv3x3_ws<64x64>", (17, 16), 64, 64, 3, 700),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_every_unit_is_computed_once(oracle, k):
    on, name, hw, cin, cout, ks, batch = CASES[k]
    rng = np.random.default_rng(88000 + k)
    b = wl._NetBuilder("order%d" % k, rng, hw[0], cin, "u8", 5, (5, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    b.conv("second", b.conv("first", 0, cout, ks, 1, ks // 2), 16, 1, 1, 0)
    x_np = wl.draw_u8(rng, (batch,) + hw + (cin,))
    x = torch.from_numpy(x_np).cuda()
    outs = []
    for switches in (on, dict(imgk=0, conv_img=0, conv_ws=0)):
        old = {n: f8.f8_tuning_get(n) for n in switches}
        try:
            for n, v in switches.items():
                f8.f8_tuning_set(n, v)
            chain = f8.Chain(b.net, keep_all=True).prepare(batch)
            assert (chain.layer_info(0, batch)[0] == name) == (switches is on), chain.layer_info(0, batch)[0]
            chain.run(x)
            outs.append(chain.tensor(b.net.layers[0].dst).clone())
        finally:
            for n, v in old.items():
                f8.f8_tuning_set(n, v)
    assert torch.equal(outs[0], outs[1])
    pick = sorted({0, batch // 2, batch - 1})
    dst = b.net.layers[0].dst
    assert np.array_equal(outs[0][pick].cpu().numpy(), oracle.run_network(b.net, np.ascontiguousarray(x_np[pick]), keep_all=True)[dst])
