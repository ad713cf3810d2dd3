"""The area-sharing kernel of the general dense path (csrc/conv_igemm.hip) against the oracle: every tile width, gathers of
16, 4 and single bytes, K at the edges of its 64-byte steps, 32-bit outputs and residuals, two formats, start values
folded by the kernel itself (single-layer calls) and taken from the chain's workspace.  Integer work: the bar is
equality."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

# B, H, W, Cin, R, S, stride, pad, x type, y type, residual, shift, dual: no layer that the LDS-direct kernel takes at
# the channel counts below
CASES = [
    (1, 1, 257, 64, 1, 1, 1, 0, "u8", "u8", None, 7, False), (1, 1, 130, 16, 1, 1, 1, 0, "s8", "s8", "s32", 5, False),
    (2, 9, 8, 80, 3, 3, 2, 1, "u8", "s32", "s32", 0, False), (1, 7, 19, 48, 3, 3, 1, 1, "u8", "u8", "s8", -2, True),
    (2, 9, 15, 4, 3, 3, 1, 1, "u8", "u8", "u8", 5, False), (3, 10, 9, 12, 5, 3, 2, 2, "s8", "u8", None, 6, True),
    (1, 1, 300, 60, 1, 1, 1, 0, "u8", "s32", None, 0, False), (2, 17, 16, 3, 3, 3, 2, 1, "u8", "u8", None, 5, False),
    (1, 13, 21, 1, 5, 5, 1, 2, "s8", "s8", "u8", 4, False), (1, 1, 259, 65, 1, 1, 1, 0, "u8", "s32", "u8", 0, False),
    (2, 12, 11, 7, 3, 3, 1, 1, "u8", "u8", None, 6, False),
]


@pytest.fixture
def area_sharing():
    f8.f8_tuning_set("wavek", 0)
    yield
    f8.f8_tuning_set("wavek", 1)


@pytest.mark.parametrize("N", [3, 16, 17, 33, 70, 131])
def test_every_tile_width_of_the_area_sharing_kernel(oracle, area_sharing, N):
    for k, (B, H, W, C, R, S, st, pd, xt, yt, rt, shift, dual) in enumerate(CASES):
        if N == 16 and rt != "s32" and C % 16 == 0:
            continue                                             # the LDS-direct kernel's
        rng = np.random.default_rng(8000 + 100 * N + k)
        x, L, res = wl.random_conv_case(rng, B, H, W, C, N, R, S, st, pd, xt, yt, rt, shift=shift)
        what = "case %d, %d channels" % (k, N)
        x_t, w_t = torch.from_numpy(x).cuda(), torch.from_numpy(L.w).cuda()
        r_t = None if res is None else torch.from_numpy(res).cuda()
        P, Q = L.out_hw
        n = B * P * Q * N
        for bias in (L.bias, None):
            b_t = None if bias is None else torch.from_numpy(bias).cuda()
            bufs = [torch.full((n + 64,), 77, dtype=f8.TORCH_DTYPE[yt], device="cuda") for _ in range(1 + dual)]
            ys = [b[16:16 + n].view(B, P, Q, N) for b in bufs]
            if dual:
                L.fl_y2, L.y2_type, L.clip_lo2, L.clip_hi2 = L.fl_x + L.fl_w + 1, yt, L.clip_lo, L.clip_hi     # second shift -1
                want = oracle.conv2d_fixed_dual(x, L.w, bias, L, (st, st), (pd, pd), res)
                f8.f8_conv2d_fixed_dual(x_t, w_t, b_t, ys[0], ys[1], L, (st, st), (pd, pd), r_t)
            else:
                want = (oracle.conv2d_fixed(x, L.w, bias, L, (st, st), (pd, pd), res),)
                f8.f8_conv2d_fixed(x_t, w_t, b_t, ys[0], L, (st, st), (pd, pd), r_t)
            torch.cuda.synchronize()
            for y, w in zip(ys, want):
                got = y.cpu().numpy()
                assert got.dtype == w.dtype and np.array_equal(got, w), "%s: %d of %d differ" % (what, int((got != w).sum()), w.size)
            for b in bufs:
                assert bool((b[:16] == 77).all()) and bool((b[16 + n:] == 77).all()), what + ": written outside the output"
        if rt or dual:
            continue
        # the same layer in a chain: start values folded beforehand (channels padded there to a multiple of 16 unless
        # the outputs are raw accumulators)
        want = oracle.conv2d_fixed(x, L.w, L.bias, L, (st, st), (pd, pd), res)
        L.src, L.dst, L.res = 0, 1, -1
        chain = f8.Chain(wl.Net("one", (H, W), C, xt, L.fl_x, [L])).prepare(B)
        if N % 4:
            assert chain.layer_info(0, B)[0].startswith("conv_igemm<"), what
        assert np.array_equal(chain.run(x_t).cpu().numpy(), want), what + ", chain"
