"""The image-stationary 3x3 kernel whose waves share K (csrc/conv_imgk.hip), forced with 1, 2 and 4 waves sharing K
on whole images, several images per workgroup (the last one partly empty), bands of rows and the smallest and
widest images, with and without residual, against the oracle.  Integer work: the bar is equality."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# C, B, H, W, x type, first y type, second y type, residual scale relative to the accumulator (None: no residual)
CASES = [
    (64, 2, 56, 56, "u8", "u8", "u8", 1), (64, 3, 11, 61, "s8", "u8", "s8", None), (64, 5, 9, 17, "u8", "s8", "u8", -1),
    (64, 7, 2, 3, "u8", "u8", "u8", 0),
    (128, 2, 28, 28, "u8", "u8", "u8", 2), (128, 3, 5, 30, "s8", "u8", "s8", None), (128, 2, 23, 17, "u8", "s8", "u8", -1),
    (128, 5, 3, 2, "u8", "u8", "u8", 0), (128, 1, 1, 1, "s8", "s8", "u8", 3),
    (256, 2, 14, 14, "u8", "u8", "u8", 1), (256, 6, 7, 7, "u8", "s8", "u8", -2), (256, 1, 21, 14, "s8", "u8", "s8", None),
    (256, 3, 2, 9, "u8", "u8", "s8", 2),
    (512, 3, 7, 7, "u8", "u8", "u8", 2), (512, 2, 8, 8, "s8", "s8", "s8", None), (512, 1, 19, 6, "u8", "u8", "u8", -1),
    (512, 4, 1, 3, "u8", "u8", "s8", 0),
]


@pytest.mark.parametrize("wk", [1, 2, 4])
def test_image_stationary_3x3_with_shared_k(oracle, wk):
    for k, (C, B, H, W, xt, yt, yt2, rd) in enumerate(CASES):
        if wk > {64: 1, 128: 2}.get(C, 4):
            continue
        rng = np.random.default_rng(9000 + k)
        x, L1, _ = wl.random_conv_case(rng, B, H, W, C, C, 3, 3, 1, 1, xt, yt, None, shift=8)
        _, L2, _ = wl.random_conv_case(rng, 1, H, W, C, C, 3, 3, 1, 1, yt, yt2, None, shift=9)
        # the second layer reads the first one's output and, as residual, the network's input
        L1.src, L1.dst, L1.res = 0, 1, -1
        L2.src, L2.dst, L2.res = 1, 2, -1
        L2.fl_x = L1.fl_y
        L2.fl_y = L2.fl_x + L2.fl_w - 9
        if rd is not None:
            L2.res, L2.res_type = 0, xt
            L2.fl_w = L1.fl_x + rd - L2.fl_x          # residual scale: fl_x + fl_w - fl_res = rd
            L2.fl_res = L1.fl_x
            L2.fl_y = L2.fl_x + L2.fl_w - 9
        net = wl.Net("imgk", (H, W), C, xt, L1.fl_x, [L1, L2])
        want = oracle.run_network(net, x, keep_all=True)
        f8.f8_tuning_set("imgk", 10 + wk)
        try:
            chain = f8.Chain(net, keep_all=True).prepare(B)
            assert [chain.layer_info(i, B)[0] for i in range(2)] == ["conv3x3_imgk<%d>" % C] * 2
            out = chain.run(torch.from_numpy(x).cuda())
            torch.cuda.synchronize()
        finally:
            f8.f8_tuning_set("imgk", 1)
        for got, w, what in ((chain.tensor(1), want[1], "first"), (out, want[2], "second")):
            got = got.cpu().numpy()
            assert got.dtype == w.dtype and np.array_equal(got, w), "case %d, %d waves, %s layer: %d of %d differ" % (
                k, wk, what, int((got != w).sum()), w.size)
        assert len(np.unique(want[2])) > 4 or want[2].size < 200, "degenerate draw"


def test_waves_sharing_k_follow_the_batch():
    """ResNet-18's 3x3 stride-1 layers take the kernel at batch 64 and (but for the two 64-channel ones without
    residual) 128, none at batch 1; images that leave most of a workgroup's pixels empty do not."""
    _, net = wl.config3(batch=1)
    f8.f8_tuning_set("conv_pair", 0)         # (two such layers in one launch are another kernel)
    try:
        chain = f8.Chain(net)
    finally:
        f8.f8_tuning_set("conv_pair", 1)

    def count(batch):
        return sum(chain.layer_info(i, batch)[0].startswith("conv3x3_imgk<") for i in range(len(net.layers)))

    assert count(1) == 0 and count(64) == 13 and count(128) == 11
    _, small = wl.config3(batch=1, hw=32)
    assert not any(f8.Chain(small).layer_info(i, 300)[0] == "conv3x3_imgk<64>" for i in range(len(small.layers)))


def test_copies_of_weights_for_the_halves_of_a_batch(oracle, always_halves):
    """401 images of 24 x 24 x 64: the whole batch does not take the kernel, its halves on two streams do."""
    rng = np.random.default_rng(5)
    b = wl._NetBuilder("halves", rng, 24, 64, "u8", 5, (5, 9), (2, 6), True)
    b.conv("second", b.conv("first", 0, 64, 3, 1, 1), 64, 3, 1, 1)
    x = wl.draw_u8(rng, (401, 24, 24, 64))
    x_t = torch.from_numpy(x).cuda()
    whole = f8.Chain(b.net).prepare(401)
    assert not whole.layer_info(0, 401)[0].startswith("conv3x3_imgk") and whole.layer_info(0, 200)[0] == "conv3x3_imgk<64>"
    halves = f8.Chain(b.net, streams=2).prepare(401)
    assert halves.streams_at(401) == 2
    got = halves.run(x_t)
    assert torch.equal(got, whole.run(x_t))
    pick = [0, 1, 199, 200, 201, 400]
    assert np.array_equal(got[pick].cpu().numpy(), oracle.run_network(b.net, np.ascontiguousarray(x[pick])))
    later = f8.Chain(b.net).prepare(401)                # two streams switched on after the workspace was made
    f8.lib().f8_chain_set_streams(later.handle, 2)
    assert later.streams_at(401) == 2
    assert torch.equal(later.run(x_t), got)


# (bands of 4 rows; of 7; of 6, the last of 5; of 3, the last of one)
@pytest.mark.parametrize("case", [(16, 56, 56, "u8", "u8", None), (45, 28, 31, "s8", "s8", "u8"), (37, 29, 31, "s8", "u8", "s8"),
                                  (13, 61, 62, "u8", "u8", "s8")])
def test_single_call_of_the_64_channel_layer_folds_itself(oracle, case):
    """f8_conv2d_fixed on 64 -> 64 channels: weights as they are, with and without bias, one launch."""
    B, H, W, xt, yt, rt = case
    rng = np.random.default_rng(77 + B)
    x, L, res = wl.random_conv_case(rng, B, H, W, 64, 64, 3, 3, 1, 1, xt, yt, rt, shift=8)
    x_t, w_t = torch.from_numpy(x).cuda(), torch.from_numpy(L.w).cuda()
    r_t = None if res is None else torch.from_numpy(res).cuda()
    for bias in (L.bias, None):
        want = oracle.conv2d_fixed(x, L.w, bias, L, (1, 1), (1, 1), res)
        y = torch.full(want.shape, 77, dtype=f8.TORCH_DTYPE[yt], device="cuda")
        f8.f8_conv2d_fixed(x_t, w_t, None if bias is None else torch.from_numpy(bias).cuda(), y, L, (1, 1), (1, 1), r_t)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want), case
    # it is this kernel that takes the call: no start values are written to scratch, unless it is switched off
    for on in (0, 1):
        f8.f8_tuning_set("imgk", on)
        n = f8.lib().f8_conv_workspace_bytes(64)
        ws = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = ws[(-ws.data_ptr()) % 256:][:n]
        f8.f8_conv2d_fixed_ws(x_t, w_t, None, y, L, ws, (1, 1), (1, 1), r_t)
        torch.cuda.synchronize()
        assert bool((ws == 0xA5).all()) == bool(on), (case, on)
        assert np.array_equal(y.cpu().numpy(), want), (case, on)
