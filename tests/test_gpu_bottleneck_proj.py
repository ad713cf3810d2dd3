"""The first block of a stage in one launch: the projection whose result is the closing layer's residual, the 3x3 layer, the closing layer and the
1x1 layer behind it, against the layers apart and the oracle."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

# channels, block's input, batch, stride, block input / projection signed, second format, projection in front of the block's first layer
CASES = [
    (64, (56, 56), 3, 1, False, True, False, True), (64, (7, 9), 11, 1, True, False, True, False), (64, (1, 3), 50, 1, False, True, True, True),
    (128, (56, 56), 2, 2, False, True, False, True), (128, (29, 31), 3, 2, True, True, True, False), (128, (3, 2), 1, 2, False, False, False, True),
    (256, (28, 28), 2, 2, False, True, True, True), (256, (13, 9), 5, 2, True, False, False, False), (256, (1, 1), 33, 2, False, True, False, True),
    (128, (14, 15), 4, 1, False, True, False, True),
]


def build(k, C, hw, stride, x_signed, p_signed, dual, first, second_reader=False):
    rng = np.random.default_rng(37000 + k)
    b = wl._NetBuilder("first%d" % k, rng, hw[0], 32, "u8", 5, (6, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    x = b.conv("x", 0, C if C == 64 else 2 * C, 1, 1, 0, relu=not x_signed)
    s = b.conv("proj", x, 4 * C, 1, stride, 0, relu=not p_signed) if first else -1
    a = b.conv("a", x, C, 1, 1, 0)
    if not first:
        s = b.conv("proj", x, 4 * C, 1, stride, 0, relu=not p_signed)
    m = b.conv("mid", a, C, 3, stride, 1)
    h = b.conv("close", m, 4 * C, 1, 1, 0, res=s, dual=dual)
    h, h2 = h if dual else (h, h)
    t = b.conv("behind", h, C, 1, 1, 0)
    e = b.conv("other", s if second_reader else h2, 32, 1, 1, 0, relu=False)
    b.conv("join", t, 32, 1, 1, 0, res=e)
    return b.net, rng


@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(CASES)))
def test_first_block_of_a_stage_in_one_launch(oracle, k):
    C, hw, batch, stride, xs, ps, dual, first = CASES[k]
    net, rng = build(k, C, hw, stride, xs, ps, dual, first)
    x = wl.draw_u8(rng, (batch,) + hw + (32,))
    want = oracle.run_network(net, x, keep_all=True)
    x_t = torch.from_numpy(x).cuda()
    names = [L.name for L in net.layers]
    try:
        for proj, force in ((0, 3), (1, 3), (1, 4)):         # the projection apart; along in the narrower and in the wider tile
            f8.f8_tuning_set("bn_proj", proj)
            f8.f8_tuning_set("bottleneck", force)
            chain = f8.Chain(net).prepare(batch)
            info = {n: chain.layer_info(i, batch)[0] for i, n in enumerate(names)}
            assert info["mid"] == "bottleneck<%d>" % C and info["close"] == info["behind"] == "(fused)"
            assert (info["proj"] == "1x1 in bottleneck<%d>" % C) == bool(proj), info
            assert all(v > 0 for v in chain.layer_info(names.index("proj"), batch)[1:])
            assert (chain.tensor(net.layers[names.index("proj")].dst) is None) == bool(proj)
            got = chain.run(x_t).cpu().numpy()
            assert np.array_equal(got, want[net.layers[-1].dst]), (CASES[k], proj, force)
            for L in net.layers[:-1]:
                for dst in (L.dst, L.dst2):
                    t = chain.tensor(dst) if dst > 0 else None
                    if t is not None:
                        assert np.array_equal(t.cpu().numpy(), want[dst]), (CASES[k], proj, force, L.name, dst)
    finally:
        f8.f8_tuning_set("bn_proj", 1)
        f8.f8_tuning_set("bottleneck", 1)


@pytest.mark.gpu
def test_projection_with_a_second_reader_stays_apart(oracle):
    net, rng = build(99, 64, (9, 9), 1, False, True, False, True, second_reader=True)
    x = wl.draw_u8(rng, (4, 9, 9, 32))
    f8.f8_tuning_set("bottleneck", 2)
    try:
        chain = f8.Chain(net).prepare(4)
        names = [chain.layer_info(i, 4)[0] for i in range(len(net.layers))]
        assert "bottleneck<64>" in names and not any(" in bottleneck" in n for n in names), names
        assert np.array_equal(chain.run(torch.from_numpy(x).cuda()).cpu().numpy(), oracle.run_network(net, x))
    finally:
        f8.f8_tuning_set("bottleneck", 1)


@pytest.mark.gpu
@pytest.mark.parametrize("private", [False, True])
def test_whole_network_with_and_without(oracle, always_halves, private):
    """ResNet-50 on 17 images: the projections along or apart, one stream and two from a captured graph: the same logits."""
    x, net = (wl.resnet50_private_fl if private else wl.config4)(batch=17, hw=96)
    x_t = torch.from_numpy(x).cuda()
    outs = []
    for proj in (0, 1):
        f8.f8_tuning_set("bn_proj", proj)
        try:
            for streams in (1, 2):
                chain = f8.Chain(net, streams=streams).prepare(17)
                assert chain.streams_at(17) == streams
                outs.append(chain.run(x_t))
                out = torch.empty_like(outs[0])
                graph = chain.capture(x_t, out)
                for _ in range(2):
                    out.zero_()
                    graph.replay()
                    torch.cuda.synchronize()
                    assert torch.equal(out, outs[0])
        finally:
            f8.f8_tuning_set("bn_proj", 1)
    assert all(torch.equal(o, outs[0]) for o in outs)
    pick = [0, 7, 8, 16]
    assert np.array_equal(outs[0][pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
