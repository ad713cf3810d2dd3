"""The streaming 1x1 kernel for 256 / 512 input channels (csrc/pw_wide.hip) in single-layer calls and chains: start values
formed from the weights it holds, second output format, every residual kind, M at the edges of its blocks of
32 pixels and of its pixel groups.  Integer work: the bar is equality."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,N,M", [(256, 1024, 2432), (256, 1024, 4097), (256, 2048, 1951), (512, 2048, 2400), (512, 512, 9631)])
def test_single_calls_of_the_wide_1x1_layers(oracle, C, N, M):
    rng = np.random.default_rng(C + N + M)
    for k, (xt, yt, rt, dual, bias) in enumerate((("u8", "u8", "u8", True, True), ("s8", "s8", "s8", True, False),
                                                  ("u8", "u8", None, True, True), ("u8", "s8", "s8", False, False))):
        x, L, res = wl.random_conv_case(rng, 1, 1, M, C, N, 1, 1, 1, 0, xt, yt, rt, shift=7)
        if rt:
            L.fl_res = L.fl_x + L.fl_w + (2 if k == 1 else -3)      # rounded right / shifted left
        b = L.bias if bias else None
        x_t, w_t = torch.from_numpy(x).cuda(), torch.from_numpy(L.w).cuda()
        b_t = None if b is None else torch.from_numpy(b).cuda()
        r_t = None if res is None else torch.from_numpy(res).cuda()
        ys = [torch.full((M * N + 64,), 77, dtype=f8.TORCH_DTYPE[yt], device="cuda") for _ in range(2)]
        y, y2 = (t[16:16 + M * N].view(1, 1, M, N) for t in ys)
        if dual:
            L.fl_y2, L.y2_type, L.clip_lo2, L.clip_hi2 = L.fl_y + (1 if k else -2), yt, L.clip_lo, L.clip_hi
            want = oracle.conv2d_fixed_dual(x, L.w, b, L, (1, 1), (0, 0), res)
            f8.f8_conv2d_fixed_dual(x_t, w_t, b_t, y, y2, L, (1, 1), (0, 0), r_t)
        else:
            want = (oracle.conv2d_fixed(x, L.w, b, L, (1, 1), (0, 0), res),)
            f8.f8_conv2d_fixed(x_t, w_t, b_t, y, L, (1, 1), (0, 0), r_t)
        torch.cuda.synchronize()
        for got, w in zip((y, y2), want):
            assert np.array_equal(got.cpu().numpy(), w), (C, N, M, k)
        for t in ys:
            assert bool((t[:16] == 77).all()) and bool((t[16 + M * N:] == 77).all())


# residual: unsigned, signed, none
@pytest.mark.parametrize("dual", [True, False])
@pytest.mark.parametrize("C,N,hw,batch,relu", [(256, 1024, 27, 23, True), (512, 2048, 9, 102, True), (256, 1024, 27, 23, False), (512, 2048, 9, 102, None)])
def test_layers_of_a_chain(oracle, C, N, hw, batch, relu, dual):
    """The same kernel behind start values from the chain's workspace, with a ragged last block."""
    rng = np.random.default_rng(C)
    b = wl._NetBuilder("dual", rng, hw, 32, "u8", 5, (5, 9), (2, 6), True)
    wide = b.conv("wide", 0, N, 1, 1, 0, relu=relu is not False)
    out = b.conv("closing", b.conv("narrow", 0, C, 1, 1, 0), N, 1, 1, 0, res=-1 if relu is None else wide, dual=dual)
    outs = out if dual else (out,)
    for t in outs:
        b.conv("reader", t, 16, 1, 1, 0)
    b.conv("last", outs[0], 16, 1, 1, 0)
    x = wl.draw_u8(rng, (batch, hw, hw, 32))
    chain = f8.Chain(b.net, keep_all=True).prepare(batch)
    assert chain.layer_info(2, batch)[0] == "pw1x1_wide<%d>" % C
    chain.run(torch.from_numpy(x).cuda())
    pick = [0, batch // 2, batch - 1]
    want = oracle.run_network(b.net, np.ascontiguousarray(x[pick]), keep_all=True)
    for t in outs:
        got = chain.tensor(t)[pick].cpu().numpy()
        assert got.dtype == want[t].dtype and np.array_equal(got, want[t]), t
