"""The K-sharing dense kernel (csrc/conv_wavek.hip) against the oracle: every tile shape forced in turn, at the
edges of tiles, K chunks, window rows and operand alignments, with the start values folded by the kernel
itself (single-layer calls) and taken from the chain's workspace.  Integer work: the bar is equality."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda"

# B, H, W, Cin, Cout, R, S, stride, pad, x type, y type, residual, shift, dual, byte offset of x
CASES = [
    # 1x1 rows: K below, at and beyond one 128-byte chunk, a last chunk that is partial, M and N at tile edges
    (1, 1, 1, 16, 4, 1, 1, 1, 0, "u8", "u8", None, 7, False, 0),
    (1, 1, 32, 128, 32, 1, 1, 1, 0, "u8", "s8", "s8", 7, False, 0),
    (1, 1, 33, 144, 36, 1, 1, 1, 0, "s8", "u8", "u8", 6, True, 0),
    (1, 1, 64, 1040, 64, 1, 1, 1, 0, "u8", "s32", None, 0, False, 0),
    (1, 1, 65, 2048, 1000, 1, 1, 1, 0, "u8", "s32", "s32", 0, False, 0),
    (3, 5, 7, 4608, 20, 1, 1, 1, 0, "u8", "u8", None, 12, False, 0),
    # windows: taps of 64 channels (two per chunk), of 128 and 192, borders, strides, non-square windows
    (2, 7, 9, 64, 64, 3, 3, 1, 1, "u8", "u8", "u8", 7, True, 0),
    (2, 8, 5, 128, 40, 3, 3, 2, 1, "u8", "s8", "s32", 8, False, 0),
    (1, 6, 6, 192, 33, 3, 3, 1, 1, "s8", "u8", None, -2, False, 0),
    (1, 9, 4, 64, 16, 5, 3, 2, 2, "u8", "u8", "s8", 5, True, 0),
    (1, 7, 7, 64, 8, 7, 7, 2, 3, "u8", "u8", None, 9, False, 0),      # more than 32 taps
    (2, 5, 5, 64, 24, 1, 1, 2, 0, "u8", "u8", None, 6, False, 0),
    # 16-byte units that are no whole 64 channels
    (2, 6, 7, 16, 12, 3, 3, 1, 1, "u8", "u8", None, 6, False, 0),
    (1, 5, 6, 80, 68, 3, 3, 2, 1, "s8", "s8", "u8", 7, False, 0),
    (1, 8, 8, 4, 8, 4, 4, 2, 0, "u8", "u8", None, 5, False, 0),       # four taps of a row per unit
    # gathered: odd channels, unaligned rows and pointers, window rows below and above 16 bytes
    (1, 1, 33, 1, 3, 1, 1, 1, 0, "u8", "u8", None, 2, False, 0),
    (2, 9, 8, 3, 10, 3, 3, 2, 1, "u8", "s8", "s8", 5, False, 0),
    (1, 6, 9, 5, 34, 3, 3, 1, 1, "s8", "u8", None, 4, True, 1),
    (2, 7, 5, 6, 66, 3, 3, 1, 1, "u8", "u8", "u8", 6, False, 3),
    (1, 11, 6, 17, 9, 5, 5, 2, 2, "u8", "s32", "s32", 0, False, 0),
    (2, 10, 13, 42, 70, 3, 3, 2, 1, "s8", "s8", None, 7, False, 0),
    (1, 5, 5, 131, 33, 1, 3, 1, 0, "u8", "u8", "s32", 8, False, 5),
    (1, 3, 3, 16, 20, 3, 3, 1, 1, "u8", "u8", None, 7, False, 4),
    (1, 2, 40, 257, 5, 1, 1, 1, 0, "s8", "u8", "u8", 9, True, 0),
]


def force(variant):
    f8.f8_tuning_set("wavek_variant", variant)


def place(a, offset):
    buf = torch.empty(a.size + 64, dtype=torch.uint8, device=DEV)
    t = buf[offset:offset + a.size].view(torch.uint8 if a.dtype == np.uint8 else torch.int8).view(*a.shape)
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("variant", range(4))
def test_every_tile_shape_of_the_k_sharing_kernel(oracle, variant):
    for k, (B, H, W, C, N, R, S, st, pd, xt, yt, rt, shift, dual, offset) in enumerate(CASES):
        rng = np.random.default_rng(7000 + k)
        x, L, res = wl.random_conv_case(rng, B, H, W, C, N, R, S, st, pd, xt, yt, rt, shift=shift)
        what = "case %d, shape %d" % (k, variant)
        args = (L, (st, st), (pd, pd), res)
        if dual:
            L.fl_y2, L.y2_type, L.clip_lo2, L.clip_hi2 = L.fl_y + (-1 if k % 2 else 1), yt, L.clip_lo, L.clip_hi
            want = oracle.conv2d_fixed_dual(x, L.w, L.bias, *args)
        else:
            want = (oracle.conv2d_fixed(x, L.w, L.bias, *args),)
        x_t, w_t, b_t = place(x, offset), torch.from_numpy(L.w).to(DEV), torch.from_numpy(L.bias).to(DEV)
        r_t = None if res is None else torch.from_numpy(res).to(DEV)
        P, Q = L.out_hw
        # outputs inside larger buffers: nothing may be written outside them
        bufs = [torch.full((B * P * Q * N + 64,), 77, dtype=f8.TORCH_DTYPE[yt], device=DEV) for _ in want]
        ys = [b[16:16 + B * P * Q * N].view(B, P, Q, N) for b in bufs]
        force(variant)
        try:
            if dual:
                f8.f8_conv2d_fixed_dual(x_t, w_t, b_t, ys[0], ys[1], L, (st, st), (pd, pd), r_t)
            else:
                f8.f8_conv2d_fixed(x_t, w_t, b_t, ys[0], L, (st, st), (pd, pd), r_t)
            torch.cuda.synchronize()
            outs = [y.cpu().numpy() for y in ys]
            if not dual and offset == 0 and yt != "s32" and not rt:
                # the same layer in a chain: start values folded beforehand
                L.src, L.dst, L.res = 0, 1, -1
                net = wl.Net("one", (H, W), C, xt, L.fl_x, [L])
                chain = f8.Chain(net).prepare(B)
                outs.append(chain.run(x_t).cpu().numpy())
                want = want + want
        finally:
            force(-1)
        for got, w in zip(outs, want):
            assert got.dtype == w.dtype and np.array_equal(got, w), "%s: %d of %d differ" % (what, int((got != w).sum()), w.size)
        for b in bufs:
            assert bool((b[:16] == 77).all()) and bool((b[16 + B * P * Q * N:] == 77).all()), what + ": written outside the output"


def test_k_sharing_kernel_is_chosen_by_size():
    """Few images take the K-sharing kernel, a large batch does not; odd channel counts with raw logits take it,
    gathering, where K is long."""
    def name(C, N, k, hw, batch, y_type="u8"):
        rng = np.random.default_rng(1)
        _, L, _ = wl.random_conv_case(rng, 1, hw, hw, C, N, k, k, 1, k // 2, "u8", y_type)
        L.src, L.dst, L.res = 0, 1, -1
        return f8.Chain(wl.Net("one", (hw, hw), C, "u8", L.fl_x, [L])).layer_info(0, batch)[0]

    assert name(512, 512, 3, 7, 1) == "conv_wavek<32x32,w8>"
    assert name(512, 128, 1, 28, 1) == "conv_wavek<32x32,w4>"
    assert name(512, 512, 3, 7, 16) == "conv_wavek<64x32,w8>"
    assert name(256, 256, 3, 14, 16) == "conv_wavek<64x64,w8>"
    assert name(2048, 512, 1, 7, 256).startswith("conv_fast<")
    assert name(301, 10, 1, 14, 256, "s32").startswith("conv_wavek_gather<")
