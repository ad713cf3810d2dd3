"""Float tensor to 8-bit codes: sizes at which a lane has two vectors, one or none, odd tails, addresses off the 16-byte grid, infinities and NaN."""
import numpy as np
import pytest
import torch

from oracle import quant_ref
from paper_2202_05239_amd import binding as f8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025, 2047, 2048, 2051, 8189, 300007])
@pytest.mark.parametrize("off", [0, 1])
def test_codes(n, off):
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n + off) * 3).astype(np.float32)
    x[off::97] = np.float32(np.inf)
    x[off + 5::101] = np.float32(-np.inf)
    t = torch.from_numpy(x).cuda()[off:]
    for fl, signed in ((5, True), (4, False)):
        got = f8.f8_fix_quant_code(t, fl, signed).cpu().numpy()
        assert np.array_equal(got.astype(np.int64), quant_ref.fix_quant_code(x[off:], fl, signed)), (n, off, signed)
    x[off] = np.nan                                        # to the lower bound
    for fl, signed in ((5, True), (4, False)):
        assert int(f8.f8_fix_quant_code(torch.from_numpy(x).cuda()[off:], fl, signed)[0]) == (-127 if signed else 0)
