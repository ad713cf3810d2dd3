"""Stride-2 3x3 layers in the image-stationary kernel, with and without the projection that reads the same input, forced with every number of
waves that share K, against the layers apart and the oracle."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# channels in, out, image, batch, input signed, projection: None, before or behind the 3x3 layer
CASES = [
    (64, 128, (56, 56), 3, False, "before"),       # bands of 7 output rows
    (64, 128, (27, 31), 5, True, "behind"),        # odd both ways: a border on the right and below
    (64, 256, (9, 62), 2, False, None),            # the widest rows; two slices of channels
    (64, 128, (5, 4), 11, False, "before"),        # several images a workgroup, the last ones missing
    (64, 128, (1, 1), 3, True, "before"), (64, 128, (61, 3), 2, False, "behind"),
    (128, 256, (28, 28), 3, False, "before"), (128, 128, (30, 11), 4, True, None), (128, 256, (2, 30), 7, False, "behind"),
    (256, 512, (14, 14), 5, False, "before"), (256, 256, (13, 9), 3, True, None), (256, 512, (7, 8), 9, False, "behind"),
]


def build(rng, cin, cout, hw, signed, where):
    b = wl._NetBuilder("s2", rng, hw[0], 16, "u8", 5, (6, 9), (2, 6), True)
    b.net.in_hw = hw
    b.t[0]["hw"] = hw
    t = b.conv("pre", 0, cin, 1, 1, 0, relu=not signed)
    d = b.conv("ds", t, cout, 1, 2, 0, relu=False) if where == "before" else -1
    a = b.conv("a", t, cout, 3, 2, 1)
    if where == "behind":
        d = b.conv("ds", t, cout, 1, 2, 0, relu=False)
    b.conv("post", a, 32, 1, 1, 0) if d < 0 else b.conv("post", a, cout, 1, 1, 0, res=d)
    return b.net


@pytest.mark.parametrize("wk", [1, 2, 4])
@pytest.mark.parametrize("k", range(len(CASES)))
def test_stride_2_layer_and_projection(oracle, k, wk):
    cin, cout, hw, batch, signed, where = CASES[k]
    if wk > {64: 1, 128: 2, 256: 4}[cin]:
        pytest.skip("no such kernel")
    rng = np.random.default_rng(61000 + k)
    net = build(rng, cin, cout, hw, signed, where)
    x = wl.draw_u8(rng, (batch,) + hw + (16,))
    x_t = torch.from_numpy(x).cuda()
    names = [L.name for L in net.layers]
    outs = []
    try:
        for mode in (0, 10 + wk):
            f8.f8_tuning_set("conv_s2", mode)
            chain = f8.Chain(net).prepare(batch)
            info = {n: chain.layer_info(i, batch)[0] for i, n in enumerate(names)}
            assert info["a"].startswith("conv3x3_imgk_s2<%d>" % cin) == (mode != 0)
            if where:
                assert info["a"].endswith("+1x1") == (mode != 0) and (info["ds"] == "(fused)") == (mode != 0)
            outs.append(chain.run(x_t))
            if mode:
                want = oracle.run_network(net, x, keep_all=True)
                for n in ("a", "ds"):
                    if n in names:
                        L = net.layers[names.index(n)]
                        got = chain.tensor(L.dst)
                        if got is not None:
                            assert np.array_equal(got.cpu().numpy(), want[L.dst]), (n, CASES[k])
                assert np.array_equal(outs[-1].cpu().numpy(), want[net.layers[-1].dst])
    finally:
        f8.f8_tuning_set("conv_s2", 1)
    assert torch.equal(outs[0], outs[1])


def test_choice_follows_the_batch():
    """ResNet-18's three stride-2 layers take their projections along at 64 images, none does at one, or at nine of 96 x 96."""
    _, net = wl.config3(batch=1)
    chain = f8.Chain(net)
    count = lambda b: sum(chain.layer_info(i, b)[0].endswith("+1x1") for i in range(len(net.layers)))
    assert count(1) == 0 and count(64) == 3 and count(192) == 3
    x, net = wl.config3(batch=9, hw=96)
    x_t = torch.from_numpy(x).cuda()
    outs = [f8.Chain(net, streams=s).prepare(9).run(x_t) for s in (1, 2)]
    outs.append(f8.Chain(net, keep_all=True).prepare(9).run(x_t))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


# ResNet-18, 96 x 96: channels of the stride-2 layers that take their projections along in the whole batch, its first half and its second
@pytest.mark.parametrize("batch, whole, low, high", [(63, [64, 256], [], [64]), (64, [64, 128, 256], [64], [64])])
def test_halves_of_a_batch_choose_for_themselves(oracle, always_halves, batch, whole, low, high):
    x, net = wl.config3(batch=batch, hw=96)
    x_t = torch.from_numpy(x).cuda()
    one, two = f8.Chain(net).prepare(batch), f8.Chain(net, streams=2).prepare(batch)
    assert two.streams_at(batch) == 2

    def taken(n):
        names = [two.layer_info(i, n)[0] for i in range(len(net.layers))]
        return [c for c in (64, 128, 256) if "conv3x3_imgk_s2<%d>+1x1" % c in names]

    assert [taken(n) for n in (batch, batch // 2, batch - batch // 2)] == [whole, low, high]
    want = one.run(x_t)
    pick = [0, batch // 2 - 1, batch // 2, batch - 1]
    assert np.array_equal(want[pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
    assert torch.equal(two.run(x_t), want) and torch.equal(f8.Chain(net, keep_all=True).prepare(batch).run(x_t), want)
    out = torch.empty_like(want)
    graph = two.capture(x_t, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(two.run(x_t), want)
