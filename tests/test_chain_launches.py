"""Launches that compute several layers of a chain: every layer is computed by exactly one of them."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl
from test_host_api import make_descs


def reported(net, batch):
    """(kernel name, operations) of every layer of the chain, switches as they stand; no GPU needed."""
    L, h, buf = f8.lib(), ctypes.c_void_p(), ctypes.create_string_buffer(64)
    ops, rows = ctypes.c_double(), []
    assert L.f8_chain_create(make_descs(net), len(net.layers), net.in_hw[0], net.in_hw[1], net.in_c, f8._TYPES[net.x_type], ctypes.byref(h)) == 0
    for i in range(len(net.layers)):
        assert L.f8_chain_layer_info(h, i, batch, buf, 64, ctypes.byref(ops), None) == 0
        rows.append((buf.value.decode(), ops.value))
    L.f8_chain_destroy(h)
    return rows


def two_readers(first, second):
    """A 3x3 128 -> 128 layer, the 1x1 layer of 512 that closes the block, and two 1x1 layers that read it."""
    rng = np.random.default_rng(61000 + first)
    b = wl._NetBuilder("two_readers", rng, 28, 16, "u8", 5, (5, 9), (2, 6), True)
    t = b.conv("mid", b.conv("before", 0, 128, 1, 1, 0), 128, 3, 1, 1)
    t = b.conv("close", t, 512, 1, 1, 0)
    u, v = b.conv("first", t, first, 1, 1, 0), b.conv("second", t, second, 1, 1, 0)
    b.conv("join", u, 32, 1, 1, 0, res=b.conv("other", v, 32, 1, 1, 0))
    return b.net, rng


@pytest.mark.parametrize("first, second", [(256, 128), (128, 256)])
def test_a_closing_layer_with_two_readers_host_side(first, second):
    """The bottleneck launch takes the first reader; the second is not the closing layer's tail then but a launch of its own."""
    net, _ = two_readers(first, second)
    for batch in (84, 100, 167):
        names = [n for n, _ in reported(net, batch)]
        assert names[1] == "bottleneck<128>" and names[2] == names[3] == "(fused)", names
        assert names[4] != "(fused)", (batch, names)


@pytest.mark.gpu
@pytest.mark.parametrize("first, second", [(256, 128), (128, 256)])
def test_a_closing_layer_with_two_readers(oracle, always_halves, first, second):
    net, rng = two_readers(first, second)
    x = wl.draw_u8(rng, (200, 28, 28, 16))
    pick = [0, 49, 99, 100, 199]
    want = oracle.run_network(net, np.ascontiguousarray(x[pick]))
    x_t = torch.from_numpy(x).cuda()
    for streams, n in ((1, 100), (2, 200)):                      # (either half of 200 images takes both launches too)
        chain = f8.Chain(net, streams=streams).prepare(n)
        assert chain.streams_at(n) == streams
        assert chain.layer_info(1, 100)[0] == "bottleneck<128>" and chain.layer_info(4, 100)[0] != "(fused)"
        got = chain.run(x_t[:n]).cpu().numpy()
        assert np.array_equal(got[[p for p in pick if p < n]], want[:sum(p < n for p in pick)])


def depthwise_projection(expand):
    """A bottleneck whose shortcut ends in a depthwise layer and the 1x1 layer behind it (with a layer in front: an inverted-residual block)."""
    rng = np.random.default_rng(66000)
    b = wl._NetBuilder("depthwise_projection", rng, 14, 16, "u8", 5, (5, 9), (2, 6), True)
    x = b.conv("x", 0, 64, 1, 1, 0)
    s = b.conv("proj", b.dwconv("dw", b.conv("expand", x, 64, 1, 1, 0) if expand else x, 3, 1, 1), 256, 1, 1, 0, relu=False)
    t = b.conv("close", b.conv("mid", b.conv("a", x, 64, 1, 1, 0), 64, 3, 1, 1), 256, 1, 1, 0, res=s)
    b.conv("after", b.conv("behind", t, 64, 1, 1, 0), 32, 1, 1, 0)
    return b.net, rng


def test_a_projection_behind_a_depthwise_layer_stays_with_it_host_side():
    """The bottleneck launch does not take a layer along that shares a launch with the layers in front of it."""
    for expand, name in ((False, "dwconv3x3<s1>+1x1"), (True, "1x1+dwconv3x3<s1>+1x1")):
        net, _ = depthwise_projection(expand)
        for batch in (1, 8, 33):
            rows = dict(zip([L.name for L in net.layers], reported(net, batch)))
            assert rows["dw"][0] == name and rows["proj"][0] == "(fused)" and rows["mid"][0] == "bottleneck<64>", (batch, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("expand", [False, True])
def test_a_projection_behind_a_depthwise_layer(oracle, expand):
    net, rng = depthwise_projection(expand)
    x = wl.draw_u8(rng, (33, 14, 14, 16))
    want = oracle.run_network(net, x)
    x_t = torch.from_numpy(x).cuda()
    for switches in (dict(), dict(dw_pw=0, pw_dw_pw=0), dict(bottleneck=4), dict(bn_proj=0), dict(bottleneck=0)):
        old = {n: f8.f8_tuning_get(n) for n in switches}
        try:
            for n, v in switches.items():
                f8.f8_tuning_set(n, v)
            for fusion in (False, True):
                got = f8.Chain(net, fusion=fusion).prepare(33).run(x_t)
                assert np.array_equal(got.cpu().numpy(), want), (switches, fusion)
        finally:
            for n, v in old.items():
                f8.f8_tuning_set(n, v)


def stage_block(c, hw):
    """The first block of a stage with the layers around it: the projection of its input, 3x3 stride 2, closing layer, the next block's first layer."""
    rng = np.random.default_rng(67000)
    b = wl._NetBuilder("stage", rng, hw, 16, "u8", 5, (5, 9), (2, 6), True)
    x = b.conv("x", 0, 2 * c, 1, 1, 0)
    s = b.conv("proj", x, 4 * c, 1, 2, 0, relu=False)
    t = b.conv("close", b.conv("mid", b.conv("a", x, c, 1, 1, 0), c, 3, 2, 1), 4 * c, 1, 1, 0, res=s)
    e = b.conv("other", t, 32, 1, 1, 0, relu=False)
    b.conv("join", b.conv("behind", t, c, 1, 1, 0), 32, 1, 1, 0, res=e)
    return b.net, rng


def places(net, batch):
    """Where the chain's tensors lie at this batch: name of the layer -> (first byte after the block's input, bytes)."""
    L, h, at = f8.lib(), ctypes.c_void_p(), ctypes.c_void_p()
    size = [ctypes.c_int() for _ in range(5)]
    assert L.f8_chain_create(make_descs(net), len(net.layers), net.in_hw[0], net.in_hw[1], net.in_c, f8._TYPES[net.x_type], ctypes.byref(h)) == 0
    rows = {}
    for S in net.layers[:-1]:
        assert L.f8_chain_tensor(h, S.dst, ctypes.c_void_p(1 << 40), batch, ctypes.byref(at), *[ctypes.byref(v) for v in size]) == 0
        if at.value:
            rows[S.name] = (at.value, batch * size[0].value * size[1].value * size[2].value)
    L.f8_chain_destroy(h)
    return {n: (a - rows["x"][0], b) for n, (a, b) in rows.items()}


def test_input_of_a_projection_lives_longer_only_where_the_launch_takes_it_along_host_side():
    """Where the projection is a launch of its own the tensors lie as if it could be nothing else; inside the bottleneck launch its input
    is not overwritten by anything that the launch writes."""
    net, _ = stage_block(256, 32)
    for batch, along in ((100, True), (128, True), (130, False), (240, False), (400, False)):
        assert (dict(zip([S.name for S in net.layers], reported(net, batch)))["proj"][0] == "1x1 in bottleneck<256>") == along
        now = places(net, batch)
        f8.f8_tuning_set("bn_proj", 0)
        try:
            apart = places(net, batch)
        finally:
            f8.f8_tuning_set("bn_proj", 1)
        assert (now == apart) == (not along), (batch, now, apart)
        for n in ("close", "behind"):
            assert not along or now[n][0] >= now["x"][1] or now[n][0] + now[n][1] <= 0, (batch, n, now)


@pytest.mark.gpu
def test_halves_that_take_a_projection_along_where_the_whole_batch_does_not(oracle):
    """3001 images: the whole batch runs the projection by itself, either half inside the bottleneck launch; streams switched after the weights
    were prepared, eager and from a captured graph."""
    net, rng = stage_block(256, 8)
    name = lambda n: dict(zip([S.name for S in net.layers], reported(net, n)))["proj"][0]
    assert name(3001) != "1x1 in bottleneck<256>" and name(1500) == name(1501) == "1x1 in bottleneck<256>"
    x = wl.draw_u8(rng, (3001, 8, 8, 16))
    x_t = torch.from_numpy(x).cuda()
    pick = [0, 1499, 1500, 3000]
    f8.f8_tuning_set("halves", 2)
    try:
        chain = f8.Chain(net).prepare(3001)
        want = chain.run(x_t)
        assert np.array_equal(want[pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
        out = torch.empty_like(want)
        for streams in (2, 1, 2):
            f8.lib().f8_chain_set_streams(chain.handle, streams)
            assert chain.streams_at(3001) == streams
            assert torch.equal(chain.run(x_t), want), streams
        graph = chain.capture(x_t, out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            assert torch.equal(chain.run(x_t), want)
    finally:
        f8.f8_tuning_set("halves", 1)


def three_in_one(rows):
    return {i for i, (n, _) in enumerate(rows) if n.startswith(("1x1+dwconv", "conv3x3+dwconv"))}


def test_switch_takes_every_block_that_fits_host_side():
    """"pw_dw_pw" = 2: the launch of three layers wherever they fit, whatever the batch and the pair's own rule say."""
    try:
        for net in (wl.mobilenet_v2_forward(batch=1)[1], wl.mobilenet_v1_forward(batch=1)[1]):
            f8.f8_tuning_set("pw_dw_pw", 2)
            f8.f8_tuning_set("dw_pw", 2)
            fits = three_in_one(reported(net, 1))
            f8.f8_tuning_set("dw_pw", 1)
            for batch in (1, 70, 256, 700):
                assert three_in_one(reported(net, batch)) == fits, (net.name, batch)
            assert fits
    finally:
        f8.f8_tuning_set("pw_dw_pw", 1)
        f8.f8_tuning_set("dw_pw", 1)


@pytest.mark.gpu
def test_switch_takes_every_block_that_fits(oracle):
    """700 images of 64 x 64: the pairs alone are two launches here, so every block reads a weight copy of its own."""
    x, net = wl.mobilenet_v2_forward(batch=700, hw=64)
    x_t = torch.from_numpy(x).cuda()
    apart = f8.Chain(net).prepare(700).run(x_t)
    f8.f8_tuning_set("pw_dw_pw", 2)
    try:
        got = f8.Chain(net).prepare(700).run(x_t)
    finally:
        f8.f8_tuning_set("pw_dw_pw", 1)
    assert torch.equal(got, apart)
    assert np.array_equal(got[[0, 699]].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[[0, 699]])))


def block(cin, ce, cout, hw, stride):
    rng = np.random.default_rng(63000)
    b = wl._NetBuilder("block", rng, hw, 16, "u8", 5, (5, 9), (2, 6), True)
    t = b.conv("before", 0, cin, 1, 1, 0, relu=False)
    y = b.conv("project", b.dwconv("dw", b.conv("expand", t, ce, 1, 1, 0), 3, stride, 1), cout, 1, 1, 0, relu=False,
               res=t if stride == 1 and cin == cout else -1)
    b.conv("after", y, 32, 1, 1, 0)
    return b.net


# (batch, expanded from, to, back to, image, stride, one launch?): microseconds of the three layers and one on either side, apart / one
RULE = [
    (120, 192, 576, 96, 33, 1, False),       # 98 / 201
    (82, 160, 480, 64, 45, 1, False),        # 107 / 195
    (15, 48, 48, 256, 93, 1, False),         # 40 / 65
    (73, 128, 384, 128, 71, 2, False),       # 108 / 143
    (14, 64, 256, 64, 83, 1, False),         # 42 / 54
    (43, 160, 960, 160, 11, 1, False),       # 25 / 29
    (73, 192, 1024, 24, 15, 2, False),       # the last two share a launch: 30 / 40
    (14, 64, 256, 32, 94, 2, True),          # 37.7 / 37.5
    (32, 80, 480, 80, 31, 1, True),          # 38 / 28
    (16, 24, 144, 24, 56, 1, True),          # MobileNetV2
    (40, 24, 144, 24, 56, 1, True),
    (64, 160, 960, 160, 7, 1, True),
    (128, 160, 960, 160, 7, 1, True),
]


@pytest.mark.parametrize("batch, cin, ce, cout, hw, stride, one", RULE)
def test_inverted_residual_launch_only_where_it_is_ahead_host_side(batch, cin, ce, cout, hw, stride, one):
    assert bool(three_in_one(reported(block(cin, ce, cout, hw, stride), batch))) == one


# (batch, channels, image, stride, channels behind, one launch?): microseconds with the layers around them, apart / one launch
BOTTLENECKS = [
    (14, 128, 78, 1, 0, False),              # 58 / 64
    (127, 64, 65, 2, 0, False),              # 52 / 60
    (60, 256, 10, 2, 0, False),              # 20.3 / 22.2
    (18, 128, 65, 2, 0, False),              # 32 / 34
    (14, 128, 78, 1, 128, True),
    (127, 64, 61, 2, 64, True),
    (60, 256, 10, 2, 256, True),
    (9, 128, 30, 1, 0, True),
]


@pytest.mark.parametrize("batch, c, hw, stride, behind, one", BOTTLENECKS)
def test_bottleneck_launch_only_where_it_is_ahead_host_side(batch, c, hw, stride, behind, one):
    """With no layer behind the closing one there is a launch less to save, and the launch stops earlier."""
    rng = np.random.default_rng(64000)
    b = wl._NetBuilder("bottleneck", rng, hw, 16, "u8", 5, (5, 9), (2, 6), True)
    y = b.conv("close", b.conv("mid", b.conv("before", 0, c, 1, 1, 0), c, 3, stride, 1), 4 * c, 1, 1, 0)
    b.conv("after", b.conv("behind", y, behind, 1, 1, 0) if behind else y, 32, 1, 1, 0)
    assert (reported(b.net, batch)[1][0] == "bottleneck<%d>" % c) == one


# (batch, channels, image, projection, one launch?): microseconds of a small forward around the layers, general kernels / this one
STRIDE_2 = [
    (64, 64, (56, 56), False, True),         # 256 workgroups: 22.4 / 20.4
    (84, 64, (52, 52), False, False),        # 336: 23.4 / 26.3
    (160, 64, (40, 40), False, False),       # 320: 24.7 / 27.7
    (160, 64, (60, 60), False, False),       # 800: 44.4 / 49.6
    (100, 64, (52, 52), True, True),         # 400: 38.9 / 36.5
    (90, 64, (56, 56), True, True),          # 360: ResNet-18 321 / 313
    (340, 64, (56, 56), True, True),         # 1360: ResNet-18 825 / 814
    (249, 128, (28, 28), True, True),        # 498: 54.4 / 50.7
    (331, 128, (49, 27), True, False),       # 1324: 100.7 / 116.8
    (121, 256, (14, 14), True, True),        # 244: 35.3 / 28.2
    (159, 256, (14, 14), True, True),        # 320: ResNet-18 471 / 464
    (198, 256, (14, 14), True, True),        # 396: 45.6 / 43.3
    (329, 256, (26, 13), True, False),       # 1316: 83.1 / 109.2
]


@pytest.mark.parametrize("batch, c, hw, projection, one", STRIDE_2)
def test_stride_2_launch_only_where_it_is_ahead_host_side(batch, c, hw, projection, one):
    b = wl._NetBuilder("stride_2", np.random.default_rng(68000), hw[0], 16, "u8", 5, (5, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    t = b.conv("before", 0, c, 1, 1, 0)
    s = b.conv("proj", t, 2 * c, 1, 2, 0, relu=False) if projection else -1
    b.conv("after", b.conv("mid", t, 2 * c, 3, 2, 1), 2 * c, 1, 1, 0, res=s)
    assert bool(taken(b.net, batch, "conv3x3_imgk_s2<%d>" % c)) == one


def test_a_launch_has_one_name_host_side():
    """The name of a layer is that of the kernel it launches, whatever kernels its layers would take apart; a layer inside another's
    launch is "(fused)"."""
    _, net = wl.mobilenet_v2_forward(batch=1)
    for batch in (1, 27, 64, 128):
        rows = reported(net, batch)
        for i in three_in_one(rows):
            kind = "conv3x3" if i == 1 else "1x1"
            assert rows[i][0] == "%s+dwconv3x3<s%d>+1x1" % (kind, net.layers[i].stride), (batch, i, rows[i])
            assert rows[i - 1] == rows[i + 1] == ("(fused)", 0.0), (batch, i)
    _, net = wl.config3(batch=1)
    rows = reported(net, 64)
    pairs = [i for i, (n, _) in enumerate(rows) if n.startswith("conv3x3_pair<")]
    assert [rows[i][0] for i in pairs] == ["conv3x3_pair<64>"] * 2 + ["conv3x3_pair<128>"]
    assert all(rows[i - 1] == ("(fused)", 0.0) for i in pairs)


def random_graph(seed):
    """A network of blocks that share launches, with the readers, shortcuts and second formats that decide whether they may."""
    rng = np.random.default_rng(62000 + seed)
    image = seed % 3 == 0
    hw = int(rng.choice((7, 14, 20, 28))) * (2 if image else 1)
    b = wl._NetBuilder("graph%d" % seed, rng, hw, 3 if image else 16, "u8", 5, (5, 9), (2, 6), True)
    yes = lambda p=0.5: bool(rng.random() < p)
    at = lambda t: b.t[t]
    loose = []                                   # second and third readers' results

    def conv(t, c, k=1, stride=1, **kw):
        return b.conv("l%d" % len(b.net.layers), t, c, k, stride, k // 2, **kw)

    def basic(t):
        c = int(rng.choice((64, 128)))
        t = t if at(t)["c"] == c else conv(t, c)
        u = conv(t, c, 3, relu=yes())
        if yes(0.15):
            loose.append(conv(u, 32))            # a second reader
        return conv(u, c, 3, res=t if yes(0.7) else -1)

    def bottleneck(t):
        c, stride = int(rng.choice((64, 128, 128, 256))), 2 if yes(0.25) and min(at(t)["hw"]) > 6 else 1
        short = conv(t, 4 * c, 1, stride) if yes() else -1
        m = conv(t if at(t)["c"] == c and yes() else conv(t, c), c, 3, stride, relu=yes(0.8))
        dual = yes(0.3)
        y = conv(m, 4 * c, res=short, relu=yes(0.8), dual=dual)
        y, y2 = y if dual else (y, y)
        readers = [conv(y if yes(0.7) else y2, int(rng.choice((c, 2 * c, c, 2 * c, 32)))) for _ in range(int(rng.integers(0, 4)))]
        loose.extend(readers[1:])
        return readers[0] if readers and yes(0.7) else y

    def inverted(t):
        stride = 2 if yes(0.3) and min(at(t)["hw"]) > 6 else 1
        u = conv(t, int(rng.choice((48, 96, 192, 384))), relu=yes(0.8)) if yes(0.8) else t
        u = b.dwconv("l%d" % len(b.net.layers), u, 3, stride, 1)
        if yes(0.1):
            loose.append(conv(u, 16))
        return conv(u, int(rng.choice((16, 24, 64, 160))), relu=yes(0.3))

    def shortcut(t):
        u = conv(t, int(rng.choice((96, 144, 192))))
        return conv(b.dwconv("l%d" % len(b.net.layers), u, 3, 1, 1), at(t)["c"], relu=False, res=t)

    t = 0
    if image:
        t = conv(0, int(rng.choice((16, 32, 64))), 3, 2)
        if at(t)["c"] <= 32 and yes(0.7):
            t = conv(b.dwconv("l1", t, 3, 1 + int(yes(0.3)), 1), int(rng.choice((16, 64))), relu=yes())
    t = conv(t, int(rng.choice((16, 64, 128)))) if yes() or t == 0 else t
    for _ in range(int(rng.integers(2, 5))):
        t = rng.choice((basic, bottleneck, bottleneck, inverted, shortcut))(t)
    last = -1
    for u in loose + [t]:                        # every branch reaches the result: pooled, then summed
        last = conv(conv(b.gpool("g%d" % len(b.net.layers), u), 32), 32, res=last)
    return b.net, rng


def operations(net, batch):
    total = 0.0
    for S in net.layers:
        if S.op in ("conv", "dwconv"):
            total += 2.0 * batch * S.out_hw[0] * S.out_hw[1] * S.R * S.S * S.Cout * (S.Cin if S.op == "conv" else 1)
    return total


@pytest.mark.parametrize("first", range(0, 120, 20))
def test_every_layer_is_computed_by_one_launch_host_side(first):
    """The operations of the reported launches add up to the network's at every batch: none is skipped, none done twice."""
    kernels = set()
    for seed in range(first, first + 20):
        net, _ = random_graph(seed)
        for batch in (1, 2, 9, 16, 50, 100, 160, 300, 500, 1200):
            rows = reported(net, batch)
            assert sum(ops for _, ops in rows) == operations(net, batch), (seed, batch, rows)
            assert all((ops == 0) == (n == "(fused)") for (n, ops), S in zip(rows, net.layers) if S.op in ("conv", "dwconv")), (seed, batch, rows)
            kernels |= {n for n, _ in rows}
    assert len(kernels) > 12


@pytest.mark.gpu
@pytest.mark.parametrize("seed", range(12))
def test_launches_of_several_layers_in_random_graphs(oracle, always_halves, seed):
    """Every tensor that is whole after a run, and the result on one stream, on two and from a captured graph, against the chain that
    keeps all tensors (layer by layer) and, for two images, against the oracle."""
    net, rng = random_graph(1000 + seed)
    batch = int(rng.choice((5, 33, 100, 201)))
    x = wl.draw_u8(rng, (batch,) + net.in_hw + (net.in_c,))
    x_t = torch.from_numpy(x).cuda()
    apart = f8.Chain(net, keep_all=True).prepare(batch)
    want = apart.run(x_t)
    pick = [0, batch - 1]
    assert np.array_equal(want[pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
    chain = f8.Chain(net).prepare(batch)
    assert torch.equal(chain.run(x_t), want), batch
    for L in net.layers[:-1]:
        for dst in (L.dst, L.dst2):
            t = chain.tensor(dst) if dst > 0 else None
            assert t is None or torch.equal(t, apart.tensor(dst)), (batch, L.name, dst)
    halves = f8.Chain(net, streams=2).prepare(batch)
    assert halves.streams_at(batch) == 2
    out = torch.empty_like(want)
    graph = halves.capture(x_t, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), batch
        assert torch.equal(halves.run(x_t), want), batch


def taken(net, batch, what):
    return [n for n, _ in reported(net, batch) if n.startswith(what)]


@pytest.mark.gpu
@pytest.mark.parametrize("C, hw, batch", [(64, 56, 24), (64, 28, 87), (128, 28, 31), (128, 28, 335)])
def test_basic_block_by_the_default_choice_on_two_streams(oracle, always_halves, C, hw, batch):
    """No switch of the launches set.  24: the whole batch takes the launch, its halves do not; 87 and 31: one of the halves does; 335: neither the whole
    batch nor its larger half does, the smaller one does (131072 pixels).  With and without a shortcut, from a captured graph too."""
    rng = np.random.default_rng(65000 + batch)
    x = wl.draw_u8(rng, (batch, hw, hw, 16))
    x_t = torch.from_numpy(x).cuda()
    pick = [0, batch // 2 - 1, batch // 2, batch - 1]
    for shortcut in (True, False):
        b = wl._NetBuilder("default", rng, hw, 16, "u8", 5, (5, 9), (2, 6), True)
        t = b.conv("before", 0, C, 1, 1, 0)
        b.conv("after", b.conv("b", b.conv("a", t, C, 3, 1, 1), C, 3, 1, 1, res=t if shortcut else -1), 32, 1, 1, 0)
        want = oracle.run_network(b.net, np.ascontiguousarray(x[pick]))
        one, two = f8.Chain(b.net).prepare(batch), f8.Chain(b.net, streams=2).prepare(batch)
        assert (one.streams_at(batch), two.streams_at(batch)) == (1, 2)
        got = one.run(x_t)
        assert np.array_equal(got[pick].cpu().numpy(), want)
        out = torch.empty_like(got)
        graph = two.capture(x_t, out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, got)
            assert torch.equal(two.run(x_t), got)


def test_basic_block_choice_host_side():
    for C, hw, batch, whole, low, high in ((64, 56, 24, 1, 0, 0), (64, 28, 87, 1, 0, 1), (128, 28, 31, 1, 0, 1), (128, 28, 335, 0, 1, 0)):
        b = wl._NetBuilder("default", np.random.default_rng(0), hw, 16, "u8", 5, (5, 9), (2, 6), True)
        t = b.conv("before", 0, C, 1, 1, 0)
        b.conv("after", b.conv("b", b.conv("a", t, C, 3, 1, 1), C, 3, 1, 1, res=t), 32, 1, 1, 0)
        count = [len(taken(b.net, n, "conv3x3_pair<%d>" % C)) for n in (batch, batch // 2, batch - batch // 2)]
        assert count == [whole, low, high], (C, hw, batch, count)


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [131, 501])
def test_inverted_residual_launches_on_halves_of_either_choice(oracle, batch):
    """MobileNetV2, 131 images: 13 launches of three layers in one half, 11 in the other, 4 in the whole batch; 501: the front's launch in one half
    only.  Two streams from a captured graph against one stream and the oracle."""
    x, net = wl.mobilenet_v2_forward(batch=batch)
    counts = [len(three_in_one(reported(net, n))) for n in (batch // 2, batch - batch // 2, batch)]
    assert counts == ([13, 11, 4] if batch == 131 else [1, 0, 0])
    x_t = torch.from_numpy(x).cuda()
    pick = [0, batch - 1]
    want = f8.Chain(net).prepare(batch).run(x_t)
    assert np.array_equal(want[pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
    chain = f8.Chain(net, streams=2).prepare(batch)
    assert chain.streams_at(batch) == 2
    out = torch.empty_like(want)
    graph = chain.capture(x_t, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(chain.run(x_t), want)
