"""Pre-processing at the edges of its kernels' strips, bands and cells: frames
smaller than a strip or a box, just past one, and wide tiles.  Whole numbers:
bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_preprocess import dev, frames, host, out_like, plan_for

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


# strips write 62 groups of four px (r <= 4) down to 56 (r 13-16); bands are 32 (u8) and 64 (u16) rows
@pytest.mark.parametrize("dtype,bits", [("u8", 8), ("u16", 12), ("u16", 16)])
@pytest.mark.parametrize("W,H,pad", [(8, 8, 0), (24, 6, 4), (246, 36, 2), (250, 64, 6), (498, 66, 2)])
@pytest.mark.parametrize("radius", [2, 3, 4, 5, 11])
def test_highpass_edges(dtype, bits, W, H, pad, radius):
    I = frames(W, H, 2, dtype, bits, 900 + W)
    I[1, ::3] = I.max()   # bright lines: the largest sums
    Id = dev(I, dtype, pad)
    out = host(plan_for(W, H, 2, dtype, bits).highpass(Id, out_like(Id, pad), radius=radius))
    for i in range(2):
        assert np.array_equal(out[i].astype(np.int64), oracle.highpass(I[i], radius)), i
