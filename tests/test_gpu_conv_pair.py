"""A basic residual block of 64 or 128 channels (3x3, 3x3, shortcut) in one launch."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# image, batch, block's input signed, first result signed, second result signed, shortcut
CASES = [
    ((56, 56), 5, False, False, False, True),
    ((28, 31), 9, True, True, False, True),        # odd width, signed shortcut
    ((61, 62), 16, False, False, True, False),      # a last band of fewer rows
    ((29, 31), 77, False, True, True, True),
    ((7, 56), 40, True, False, False, False),
    ((1, 56), 3, False, True, False, True),         # one row: a row of zeros on either side of both tensors
    ((37, 24), 18, False, False, False, True),
    ((28, 28), 7, False, False, False, True, 128),
    ((19, 28), 5, True, True, True, True, 128),
    ((30, 27), 6, False, True, False, False, 128),
    ((1, 28), 3, False, False, False, True, 128),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_basic_block_in_one_launch(oracle, k):
    hw, batch, xs, es, ys, res, C = CASES[k] if len(CASES[k]) == 7 else CASES[k] + (64,)
    rng = np.random.default_rng(54000 + k)
    b = wl._NetBuilder("basic%d" % k, rng, hw[0], 16, "u8", 5, (6, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw

    def conv(name, src, cout, ks, signed, r=-1):
        t = b.conv(name, src, cout, ks, 1, ks // 2, res=r)
        L = b.net.layers[-1]
        if signed:
            L.y_type, L.clip_lo, L.clip_hi = "s8", -127, 100
            b.t[t]["type"] = "s8"
        return t

    t = conv("before", 0, C, 1, xs)
    conv("after", conv("b", conv("a", t, C, 3, es), C, 3, ys, t if res else -1), 32, 1, False)
    net = b.net
    x = wl.draw_u8(rng, (batch,) + hw + (16,))
    x_t = torch.from_numpy(x).cuda()
    outs = {}
    try:
        for force in (0, 1):
            f8.f8_tuning_set("conv_pair", force)
            f8.f8_tuning_set("imgk", 11)
            chain = f8.Chain(net).prepare(batch)
            names = [chain.layer_info(i, batch)[0] for i in (1, 2)]
            assert names == (["conv3x3_imgk<%d>" % C] * 2 if force == 0 else ["(fused)", "conv3x3_pair<%d>" % C])
            outs[force] = chain.run(x_t)
            assert force == 0 or chain.tensor(net.layers[1].dst) is None
    finally:
        f8.f8_tuning_set("conv_pair", 1)
        f8.f8_tuning_set("imgk", 1)
    assert torch.equal(outs[0], outs[1]), (CASES[k], int((outs[0] != outs[1]).sum()))
    pick = [0, batch // 2, batch - 1]
    want = oracle.run_network(net, np.ascontiguousarray(x[pick]), keep_all=True)
    assert np.array_equal(outs[1].cpu().numpy()[pick], want[net.layers[-1].dst]), CASES[k]
    assert len(np.unique(want[net.layers[2].dst])) > 4, "degenerate draw"


def test_the_second_layer_may_open_a_bottleneck(oracle):
    """3x3, 3x3, 1x1 of four times the channels: the last three layers share a launch and read what the first one wrote."""
    rng = np.random.default_rng(54100)
    b = wl._NetBuilder("both", rng, 28, 16, "u8", 5, (6, 9), (2, 6), True)
    t = b.conv("a", b.conv("before", 0, 64, 1, 1, 0), 64, 3, 1, 1)
    b.conv("after", b.conv("c", b.conv("b", t, 64, 3, 1, 1), 256, 1, 1, 0), 64, 1, 1, 0)
    b.conv("last", len(b.t) - 1, 32, 1, 1, 0)
    x = wl.draw_u8(rng, (40, 28, 28, 16))
    f8.f8_tuning_set("imgk", 11)
    try:
        chain = f8.Chain(b.net).prepare(40)
        assert chain.layer_info(2, 40)[0] == "bottleneck<64>" and chain.layer_info(1, 40)[0] == "conv3x3_imgk<64>"
        got = chain.run(torch.from_numpy(x).cuda()).cpu().numpy()
    finally:
        f8.f8_tuning_set("imgk", 1)
    assert np.array_equal(got[:3], oracle.run_network(b.net, np.ascontiguousarray(x[:3])))
