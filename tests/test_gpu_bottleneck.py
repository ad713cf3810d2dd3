"""The 3x3 layer of a bottleneck block, the closing 1x1 layer (residual, one or two output formats) and the 1x1 layer that
opens the next block in one launch."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

# channels, image, batch, stride, channels behind (0: none), input / residual signed, second format, residual, layer between
CASES = [
    (64, (56, 56), 3, 1, 64, False, False, False, True, False),
    (64, (7, 9), 11, 1, 128, True, True, True, True, True),        # tiles over several images
    (64, (1, 3), 50, 1, 64, False, True, False, True, False),      # one-row images: 22 or more in a tile
    (64, (13, 70), 2, 2, 0, False, False, True, False, False),     # nothing behind, no residual, rows of more than one KiB
    (128, (28, 28), 2, 1, 128, False, False, True, True, False),
    (128, (29, 31), 3, 2, 256, True, False, False, True, True),    # odd extents under stride 2
    (128, (5, 3), 9, 1, 0, False, True, False, True, False),
    (128, (2, 2), 1, 1, 128, True, False, True, False, False),     # fewer pixels than a tile
    (256, (14, 14), 3, 1, 256, False, False, False, True, False),
    (256, (14, 14), 1, 1, 512, True, True, True, True, True),
    (256, (9, 11), 4, 2, 256, False, True, True, False, False),
    (256, (1, 1), 70, 1, 0, False, False, False, True, False),     # every tap but the middle one outside the image
]


def build(k, C, hw, stride, behind, signed, res_signed, dual, with_res, between):
    rng = np.random.default_rng(31000 + k)
    b = wl._NetBuilder("bottleneck%d" % k, rng, hw[0], 32, "u8", 5, (5, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    s = b.conv("short", 0, 4 * C, 1, stride, 0, relu=not res_signed)
    a = b.conv("first", 0, C, 1, 1, 0, relu=not signed)
    m = b.conv("mid", a, C, 3, stride, 1, relu=k % 3 != 1)
    h = b.conv("close", m, 4 * C, 1, 1, 0, relu=k % 4 != 3, res=s if with_res else -1, dual=dual)
    h, h2 = h if dual else (h, h)
    if between:          # the next stage's shortcut projection
        e = b.conv("other_reader", h2, 32, 1, 1, 0, relu=False)
    t = b.conv("behind", h, behind, 1, 1, 0, relu=k % 2 == 0) if behind else h
    if not between:
        e = b.conv("other_reader", h2, 32, 3, 1, 1, relu=False)
    b.conv("join", t, 32, 1 if behind else 3, 1, 0 if behind else 1, res=e)
    return b.net, wl.draw_u8(rng, (0,) + hw + (32,)), rng


@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(CASES)))
def test_three_layers_of_a_bottleneck_in_one_launch(oracle, k):
    C, hw, batch, stride, behind, signed, res_signed, dual, with_res, between = CASES[k]
    net, _, rng = build(k, C, hw, stride, behind, signed, res_signed, dual, with_res, between)
    x = wl.draw_u8(rng, (batch,) + hw + (32,))
    want = oracle.run_network(net, x, keep_all=True)
    x_t = torch.from_numpy(x).cuda()
    try:
        for force in (0, 3, 4):          # three launches; one with the narrower and with the wider tile
            f8.f8_tuning_set("bottleneck", force)
            chain = f8.Chain(net).prepare(batch)
            names = [chain.layer_info(i, batch)[0] for i in range(len(net.layers))]
            assert (names[2] == "bottleneck<%d>" % C) == (force != 0) and (names[3] == "(fused)") == (force != 0), names
            assert not behind or (names[5 if between else 4] == "(fused)") == (force != 0), names
            got = chain.run(x_t)
            torch.cuda.synchronize()
            got = got.cpu().numpy()
            assert np.array_equal(got, want[net.layers[-1].dst]), (CASES[k], force, int((got != want[net.layers[-1].dst]).sum()))
            for L in net.layers[:-1]:    # tensors that are whole after the run: the block output, its second format, the layer behind
                for dst in (L.dst, L.dst2):
                    t = chain.tensor(dst) if dst > 0 else None
                    if t is not None:
                        assert np.array_equal(t.cpu().numpy(), want[dst]), (CASES[k], force, L.name, dst)
            assert (chain.tensor(net.layers[2].dst) is None) or force == 0
    finally:
        f8.f8_tuning_set("bottleneck", 1)
    assert len(np.unique(want[net.layers[-1].dst])) > 4, "degenerate draw"


@pytest.mark.gpu
def test_blocks_in_one_launch_through_streams_and_graphs(oracle, always_halves):
    """ResNet-50 with two formats, 96 x 96 images: halves on two streams (batches that take the launch and batches that do
    not), a captured graph replayed with eager work between, against the oracle."""
    x, net = wl.resnet50_private_fl(batch=5, hw=96)
    want = oracle.run_network(net, x)
    x_t = torch.from_numpy(x).cuda()
    chain = f8.Chain(net, streams=2).prepare(5)
    assert chain.streams_at(5) == 2
    out = torch.empty((5,) + chain.out_shape, dtype=chain.out_dtype, device="cuda")
    graph = chain.capture(x_t, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
        chain.run(x_t)
    assert np.array_equal(f8.Chain(net).prepare(5).run(x_t).cpu().numpy(), want)


def test_blocks_in_one_launch_follow_the_batch_host_side():
    """ResNet-50: seven blocks of the first two stages at one image (256 channels stream too many weights for so few pixels),
    all thirteen at 16, none at 256; not where every tensor is kept; the weights' copies only where a batch needs them."""
    _, net = wl.config4(batch=1)
    L, h, n, buf = f8.lib(), ctypes.c_void_p(), ctypes.c_size_t(), ctypes.create_string_buffer(64)
    from test_host_api import make_descs
    assert L.f8_chain_create(make_descs(net), len(net.layers), 224, 224, 3, f8.F8_S8, ctypes.byref(h)) == 0

    def count(batch):
        total = 0
        for i in range(len(net.layers)):
            assert L.f8_chain_layer_info(h, i, batch, buf, 64, None, None) == 0
            total += buf.value.decode().startswith("bottleneck<")
        return total

    def size(batch):
        assert L.f8_chain_workspace_bytes(h, batch, ctypes.byref(n)) == 0
        return n.value

    assert (count(1), count(16), count(256)) == (7, 13, 0)
    sizes = [size(b) for b in range(0, 40)]
    assert sizes == sorted(sizes)
    assert L.f8_chain_set_keep_all(h, 1) == 0
    assert count(16) == 0
    L.f8_chain_destroy(h)
