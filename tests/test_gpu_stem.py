"""The 7x7 stride-2 layer on the image and the max pool behind it in one launch, on images as the caller has them."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# image, batch, unsigned image, bytes that the image's address is off the four-byte grid; up to 2048 tiles of 7 x 7 pooled pixels a
# wave takes 32 channels, beyond all 64; rows of a multiple of four pixels at a four-byte address are fetched without shifting
CASES = [
    ((28, 28), 5, True, 0), ((28, 28), 5, True, 1), ((29, 32), 3, False, 2), ((61, 57), 4, True, 3), ((57, 58), 3, False, 0), ((30, 59), 6, True, 0),
    ((1, 1), 3, True, 1), ((2, 3), 5, True, 0), ((4, 4), 2, False, 0), ((7, 200), 3, True, 0), ((130, 5), 3, True, 0),
    ((28, 28), 2048, True, 0),                     # the last size of the first kind, the first of the second
    ((28, 28), 2049, True, 0), ((26, 27), 2300, True, 1), ((29, 30), 520, False, 0), ((9, 13), 2100, False, 3),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_stem_reads_the_image_itself(oracle, k):
    hw, batch, unsigned, off = CASES[k]
    rng = np.random.default_rng(71000 + k)
    b = wl._NetBuilder("stem%d" % k, rng, hw[0], 3, "u8" if unsigned else "s8", 5, (5, 9), (2, 6), False)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    b.maxpool("pool", b.conv("conv1", 0, 64, 7, 2, 3))
    net = b.net
    n = batch * hw[0] * hw[1] * 3
    # bytes of the whole range around the image too: none of them may reach a result
    buf = torch.from_numpy(rng.integers(0, 256, n + 16).astype(np.uint8)).cuda()
    x_t = buf[off:off + n].view(torch.uint8 if unsigned else torch.int8).reshape((batch,) + hw + (3,))
    assert x_t.data_ptr() % 4 == off
    chain = f8.Chain(net).prepare(batch)
    assert chain.layer_info(0, batch)[0] == "stem_pool_fused"
    got = chain.run(x_t)
    apart = f8.Chain(net, keep_all=True).prepare(batch)
    assert torch.equal(got, apart.run(x_t))
    some = sorted({0, batch // 2, batch - 1})
    assert np.array_equal(got.cpu().numpy()[some], oracle.run_network(net, x_t.cpu().numpy()[some]))


@pytest.mark.parametrize("hw", [(1, 11_500_000), (1, 11_500_003), (2, 5_700_001), (11_500_001, 1)])
def test_images_of_a_few_rows_or_columns(oracle, hw):
    """The bytes of the image are what has to be addressable, whatever its shape; both ends against the oracle on a piece of the image."""
    rng = np.random.default_rng(72000 + hw[0])
    b = wl._NetBuilder("thin", rng, hw[0], 3, "u8", 5, (5, 9), (2, 6), False)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    b.maxpool("pool", b.conv("conv1", 0, 64, 7, 2, 3))
    x = wl.draw_u8(rng, (1,) + hw + (3,))
    x_t = torch.from_numpy(x).cuda()
    chain = f8.Chain(b.net).prepare(1)
    assert chain.layer_info(0, 1)[0] == "stem_pool_fused"
    got = chain.run(x_t)
    apart = f8.Chain(b.net, keep_all=True).prepare(1)
    assert torch.equal(got, apart.run(x_t))
    n, axis = max(hw), 1 if hw[0] > hw[1] else 2
    for first in (0, (n - 400) // 4 * 4):                # (two strides of two)
        piece = np.ascontiguousarray(np.take(x, range(first, min(n, first + 403)), axis=axis))
        size = piece.shape[1:3]
        p = wl._NetBuilder("piece", rng, size[0], 3, "u8", 5, (5, 9), (2, 6), False)
        p.net.in_hw = size
        p.t[0]["hw"] = size
        p.maxpool("pool", p.conv("conv1", 0, 64, 7, 2, 3))
        for L, K in zip(p.net.layers, b.net.layers):
            L.w, L.bias, L.fl_x, L.fl_w, L.fl_y, L.clip_lo, L.clip_hi = K.w, K.bias, K.fl_x, K.fl_w, K.fl_y, K.clip_lo, K.clip_hi
        want = oracle.run_network(p.net, piece)
        # (without the outputs whose window reaches over the cut)
        lo, hi = (0, 95) if first == 0 else (5, want.shape[axis])
        mine = got[:, first // 4:first // 4 + hi] if axis == 1 else got[:, :, first // 4:first // 4 + hi]
        take = (slice(None), slice(lo, hi)) if axis == 1 else (slice(None), slice(None), slice(lo, hi))
        assert np.array_equal(mine.cpu().numpy()[take], want[take]), (hw, first)
