"""The image-stationary 3x3 kernel with single and twice the waves: on either side of the line between the two, last bands and images missing,
against the general kernel and, for a few images, the oracle; single calls of 64 channels on either side of theirs."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# channels, image, waves that share K, batch
CASES = [(64, (56, 56), 1, 1024 // 14), (64, (56, 56), 1, 1024 // 14 + 1), (64, (56, 56), 1, 2048 // 14), (64, (56, 56), 1, 2048 // 14 + 1), (64, (5, 61), 1, 3), (64, (1, 1), 1, 2),
         (128, (28, 28), 1, 64), (128, (28, 28), 1, 65), (128, (9, 30), 2, 5), (256, (14, 14), 2, 64), (256, (14, 14), 2, 65), (256, (14, 14), 4, 32),
         (256, (3, 5), 4, 9), (512, (7, 7), 4, 31), (512, (7, 7), 2, 65), (512, (7, 7), 1, 5)]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_single_and_twice_the_waves(oracle, k):
    C, hw, wk, batch = CASES[k]
    rng = np.random.default_rng(93000 + k)
    b = wl._NetBuilder("waves%d" % k, rng, hw[0], C, "u8", 5, (6, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    b.conv("second", b.conv("first", 0, C, 3, 1, 1), C, 3, 1, 1, res=0)
    x_np = wl.draw_u8(rng, (batch,) + hw + (C,))
    x = torch.from_numpy(x_np).cuda()
    outs = []
    try:
        for mode in (10 + wk, 0):
            f8.f8_tuning_set("imgk", mode)
            f8.f8_tuning_set("conv_img", 0)
            chain = f8.Chain(b.net, keep_all=True).prepare(batch)
            assert (chain.layer_info(0, batch)[0] == "conv3x3_imgk<%d>" % C) == (mode != 0)
            outs.append((chain.run(x), chain.tensor(1).clone()))
    finally:
        f8.f8_tuning_set("imgk", 1)
        f8.f8_tuning_set("conv_img", 1)
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    pick = sorted({0, batch // 2, batch - 1})
    want = oracle.run_network(b.net, np.ascontiguousarray(x_np[pick]), keep_all=True)
    for got, dst in zip(outs[0], (b.net.layers[-1].dst, 1)):
        assert np.array_equal(got[pick].cpu().numpy(), want[dst])


@pytest.mark.parametrize("batch", [3, 4, 36, 37])
def test_single_call_weights_through_lds(oracle, batch):
    rng = np.random.default_rng(95000 + batch)
    x, L, res = wl.random_conv_case(rng, batch, 56, 56, 64, 64, 3, 3, 1, 1, "u8", "u8", "s8", shift=8)
    y = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    dev = [torch.from_numpy(a).cuda() for a in (x, L.w, L.bias, res)]
    f8.f8_conv2d_fixed(dev[0], dev[1], dev[2], y, L, (1, 1), (1, 1), dev[3])
    some = sorted({0, batch // 2, batch - 1})
    assert np.array_equal(y.cpu().numpy()[some], oracle.conv2d_fixed(x[some], L.w, L.bias, L, (1, 1), (1, 1), res[some]))
