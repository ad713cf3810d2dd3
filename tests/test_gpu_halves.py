"""Two streams: the halves of a small batch side by side where that is asked for (tuning switch), one stream by the default choice, the same results;
a batch on the other side of the line."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

NETS = [(wl.config4, 5, 96), (wl.resnet50_private_fl, 5, 96), (wl.config3, 24, 96), (wl.mobilenet_v2_forward, 11, 96), (wl.mobilenet_v1_forward, 3, 64),
        (wl.config3, 65, 224)]


def test_batch_that_needs_more_launches_than_its_halves():
    """Below the line too the halves run side by side where the whole batch is several launches more: MobileNetV2's blocks from 32 images on."""
    _, net = wl.mobilenet_v2_forward(batch=1)
    two, one = f8.Chain(net, streams=2), f8.Chain(net)

    def launches(n):
        return sum(two.layer_info(i, n)[0] != "(fused)" for i in range(len(net.layers)))

    for n in (11, 27, 30, 39, 41, 43):
        assert (two.streams_at(n) == 2) == (launches(n) >= launches(n - n // 2) + 4), n
        assert one.streams_at(n) == 1
    assert two.streams_at(27) == 1 and two.streams_at(41) == 2
    x = torch.from_numpy(wl.mobilenet_v2_forward(batch=41)[0]).cuda()
    assert torch.equal(two.prepare(41).run(x), one.prepare(41).run(x))


@pytest.mark.parametrize("k", range(len(NETS)))
def test_halves_side_by_side_or_not(oracle, k):
    fn, batch, hw = NETS[k]
    long_enough = hw == 224                   # (the line: 15 images of ResNet-18 at 224 x 224, far above the batches of the small images)
    x, net = fn(batch=batch, hw=hw)
    x_t = torch.from_numpy(x).cuda()
    want = f8.Chain(net).prepare(batch).run(x_t)
    pick = sorted({0, batch // 2, batch - 1})
    assert np.array_equal(want[pick].cpu().numpy(), oracle.run_network(net, np.ascontiguousarray(x[pick])))
    try:
        for mode in (1, 2):
            f8.f8_tuning_set("halves", mode)
            chain = f8.Chain(net, streams=2).prepare(batch)
            assert chain.streams_at(batch) == (2 if mode == 2 or long_enough else 1)
            out = torch.empty_like(want)
            graph = chain.capture(x_t, out)
            for _ in range(3):
                out.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, want), (mode, "graph")
                assert torch.equal(chain.run(x_t), want), mode
            # tensors inside a chain on two streams are not reported, whichever way it runs
            assert all(chain.tensor(L.dst) is None for L in net.layers[:-1])
    finally:
        f8.f8_tuning_set("halves", 1)
