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


# the mapping pass by cells (power-of-two tiles, ragged ones, one tile, cells
# narrower than a group of four pixels, wide u16 blends) and the pass for small u8 tiles
@pytest.mark.parametrize("dtype,bits,W,H,pad,tiles", [
    ("u8", 8, 256, 256, 0, (4, 2)), ("u8", 8, 250, 130, 6, (3, 5)), ("u8", 8, 198, 138, 2, (1, 1)),
    ("u8", 8, 1200, 40, 4, (1, 1)), ("u8", 8, 4096, 64, 0, (1, 2)), ("u8", 8, 64, 64, 0, (16, 16)),
    ("u8", 8, 96, 96, 4, (2, 30)), ("u16", 12, 250, 130, 2, (7, 5)), ("u16", 12, 64, 48, 0, (40, 31)),
    ("u16", 12, 48, 24, 0, (16, 8)), ("u16", 12, 1536, 1152, 0, (2, 1)), ("u16", 16, 250, 130, 2, (4, 3)),
    ("u16", 16, 640, 480, 0, (2, 1)), ("u16", 16, 512, 96, 2, (2, 48))])
def test_clahe_cells(dtype, bits, W, H, pad, tiles):
    I = frames(W, H, 2, dtype, bits, 700 + W)
    I[1] = np.random.default_rng(W).integers(0, 1 << bits, (H, W))   # every bin, the largest blends
    P = plan_for(W, H, 2, dtype, bits)
    Id = dev(I, dtype, pad)
    full = Id._base if Id._base is not None else Id
    out = host(P.clahe(Id, out_like(Id, pad), tiles=tiles, clip_factor=2.5))
    ref = np.stack([oracle.clahe(I[i], bits, tiles[0], tiles[1], 2.5) for i in range(2)])
    assert np.array_equal(out.astype(np.int64), ref.astype(np.int64))
    P.clahe(Id, Id, tiles=tiles, clip_factor=2.5)   # in place, the padding left alone
    assert np.array_equal(host(Id).astype(np.int64), ref.astype(np.int64))
    if pad:
        assert (host(full)[:, :, W:] == np.iinfo(I.dtype).max).all()


# histograms of tiles that begin and end anywhere in a word, narrower than a
# word, than the four words of a read, and with one to five words at the sides
@pytest.mark.parametrize("dtype,bits", [("u8", 8), ("u16", 12)])
@pytest.mark.parametrize("W,tiles_x", [(46, 46), (46, 13), (46, 2), (130, 7), (150, 4), (198, 7), (198, 1), (202, 3)])
def test_clahe_tile_sides(dtype, bits, W, tiles_x):
    I = np.random.default_rng(W + tiles_x).integers(0, 1 << bits, (2, 22, W)).astype(np.uint8 if dtype == "u8" else np.uint16)
    I[:, ::2, ::3] = 0
    Id = dev(I, dtype, 2)
    out = host(plan_for(W, 22, 2, dtype, bits).clahe(Id, out_like(Id, 2), tiles=(tiles_x, 2), clip_factor=3.0))
    ref = np.stack([oracle.clahe(I[i], bits, tiles_x, 2, 3.0) for i in range(2)])
    assert np.array_equal(out.astype(np.int64), ref.astype(np.int64))
