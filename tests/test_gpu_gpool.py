"""Global pool on either side of the line between its two kernels: few pixels, many workgroups, channels that fill no workgroup, signed
tensors, raw sums, negative shifts."""
import numpy as np
import pytest
import torch

from paper_2202_05239_amd import binding as f8
from paper_2202_05239_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [((3, 7, 7, 2048), "u8", "u8", 6), ((2, 5, 5, 260), "s8", "s8", 5), ((2, 4, 6, 256), "u8", "u8", 5), ((1, 25, 1, 4), "u8", "s32", 5), ((5, 9, 13, 12), "s8", "s8", -1),
         ((768, 5, 5, 128), "u8", "u8", 5), ((769, 5, 5, 128), "u8", "u8", 5), ((2, 61, 53, 516), "u8", "u8", 12), ((3, 7, 7, 30), "u8", "u8", 6)]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_global_pool(oracle, k):
    shape, xt, yt, shift = CASES[k]
    rng = np.random.default_rng(41000 + k)
    x = rng.integers(0, 256, shape).astype(np.uint8) if xt == "u8" else rng.integers(-128, 128, shape).astype(np.int8)
    fl_w = 6
    L = wl.LayerSpec(op="gpool", Cin=shape[3], Cout=shape[3], fl_x=4, fl_w=fl_w, fl_y=4 + fl_w - shift, clip_lo=-127 if yt == "s8" else 0,
                     clip_hi=127 if yt == "s8" else 255, x_type=xt, y_type=yt, in_hw=shape[1:3], out_hw=(1, 1))
    want = oracle.global_pool_fixed(x, L)
    y = torch.empty(want.shape, dtype=f8.TORCH_DTYPE[yt], device="cuda")
    f8.f8_global_pool_fixed(torch.from_numpy(x).cuda(), y, L)
    assert np.array_equal(y.cpu().numpy(), want)
