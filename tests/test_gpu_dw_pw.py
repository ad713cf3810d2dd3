"""A depthwise 3x3 layer and the 1x1 layer behind it in one launch (csrc/dw_pw.hip), forced at any batch: both strides,
rows from one pixel to 128, the last tile of an image partly empty, K ending in half a slice, every number of waves sharing
K, with and without residual, signed and unsigned tensors, against the oracle.  Integer work: the bar is equality."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# stride, B, H, W, C, N, input type, depthwise output type, output type, residual scale relative to the accumulator (None: none)
CASES = [
    (1, 2, 112, 112, 32, 16, "u8", "u8", "s8", None), (1, 1, 5, 128, 16, 8, "s8", "u8", "u8", 0), (1, 1, 9, 65, 48, 24, "u8", "s8", "s8", 2),
    (1, 3, 28, 28, 144, 32, "u8", "u8", "s8", 1), (1, 2, 14, 14, 576, 96, "u8", "u8", "s8", -1), (1, 4, 7, 7, 960, 160, "u8", "u8", "s8", 2),
    (1, 2, 7, 7, 1024, 256, "s8", "s8", "u8", None), (1, 5, 1, 1, 80, 40, "u8", "u8", "u8", -2), (1, 300, 3, 2, 112, 200, "s8", "u8", "s8", 1),
    (1, 260, 9, 8, 64, 104, "u8", "u8", "u8", None),
    (2, 2, 112, 112, 96, 24, "u8", "u8", "s8", None), (2, 3, 55, 57, 144, 32, "s8", "u8", "u8", None), (2, 1, 7, 255, 16, 72, "u8", "s8", "u8", None),
    (2, 4, 14, 14, 176, 160, "u8", "u8", "s8", None), (2, 200, 15, 13, 240, 256, "u8", "u8", "u8", None), (2, 2, 1, 1, 32, 8, "u8", "u8", "u8", None),
    (2, 3, 2, 5, 528, 64, "s8", "s8", "s8", None),
]


def pair(k, case):
    """1x1 layer N -> C, the depthwise one, 1x1 layer C -> N (with the network's input as residual): (x, net)"""
    stride, B, H, W, C, N, xt, dt, yt, rd = case
    rng = np.random.default_rng(4100 + k)
    x, L0, _ = wl.random_conv_case(rng, B, H, W, N, C, 1, 1, 1, 0, xt, xt, None, shift=6)
    _, L1, _ = wl.random_conv_case(rng, 1, H, W, C, C, 3, 3, stride, 1, xt, dt, None, shift=5, depthwise=True)
    _, L2, _ = wl.random_conv_case(rng, 1, L1.out_hw[0], L1.out_hw[1], C, N, 1, 1, 1, 0, dt, yt, None, shift=7)
    for i, (L, s) in enumerate(((L0, 6), (L1, 5), (L2, 7))):
        L.src, L.dst, L.res = i, i + 1, -1
        if i:
            L.fl_x = (L0, L1)[i - 1].fl_y
        if i == 2 and rd is not None:
            L.res, L.res_type, L.fl_res = 0, xt, L0.fl_x
            L.fl_w = L0.fl_x + rd - L.fl_x
        L.fl_y = L.fl_x + L.fl_w - s
    return x, wl.Net("pair", (H, W), N, xt, L0.fl_x, [L0, L1, L2])


@pytest.mark.parametrize("k", range(len(CASES)))
def test_depthwise_and_1x1_in_one_launch(oracle, k):
    case = CASES[k]
    x, net = pair(k, case)
    B = case[1]
    if k % 3 == 1:
        net.layers[1].bias = None
    want = oracle.run_network(net, x)
    x_t = torch.from_numpy(x).cuda()
    for force, behind in ((2, "dwconv3x3<s%d>+1x1" % case[0]), (0, "dwconv3x3<s%d>" % case[0])):
        f8.f8_tuning_set("dw_pw", force)
        try:
            chain = f8.Chain(net).prepare(B)
        finally:
            f8.f8_tuning_set("dw_pw", 1)
        assert chain.layer_info(1, B)[0] == behind and (chain.layer_info(2, B)[0] == "(fused)") == (force == 2)
        for _ in range(2):
            got = chain.run(x_t).cpu().numpy()
            assert got.dtype == want.dtype and np.array_equal(got, want), (case, force, int((got != want).sum()), want.size)
    assert len(np.unique(want)) > 4 or want.size < 200, "degenerate draw"


def test_output_at_an_odd_address_runs_the_two_layers(oracle):
    x, net = pair(3, CASES[3])
    B = CASES[3][1]
    want = oracle.run_network(net, x)
    chain = f8.Chain(net).prepare(B)
    assert chain.layer_info(2, B)[0] == "(fused)"
    room = torch.full((want.size + 16,), 77, dtype=f8.TORCH_DTYPE["s8"], device="cuda")
    for off in (0, 4, 1):
        out = room[off:off + want.size].view(want.shape)
        chain.run(torch.from_numpy(x).cuda(), out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), off


def test_pairs_follow_the_batch():
    """MobileNetV2's depthwise layers share a launch with the 1x1 layer behind them at batch 1 (but for the three with
    960 channels), none does at batch 256."""
    _, net = wl.mobilenet_v2_forward(batch=1)
    f8.f8_tuning_set("pw_dw_pw", 0)          # (pairs that are part of a larger launch do not show)
    try:
        chain = f8.Chain(net)
    finally:
        f8.f8_tuning_set("pw_dw_pw", 1)

    def count(batch):
        return sum("+1x1" in chain.layer_info(i, batch)[0] for i in range(len(net.layers)))

    assert count(1) == 14 and count(27) == 11 and count(256) == 0
