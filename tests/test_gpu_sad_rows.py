"""The 2x2-cell block searches against the integer oracle, bit for bit, where
a wave's parents run over the end of a grid row: odd grids, grids narrower
than a wave, one row or column of parents, and every coarse radius (whose last
pass of shift rows is shorter)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# dtype, grid, levels, radius_coarse, radius_fine
# (few tiles: a workgroup per 21 parents; 20 pairs: a wave)
CASES = [("u8", g, 2, rc, rf) for g in ((43, 27), (85, 3), (3, 44), (22, 21), (42, 42)) for rc, rf in ((3, 1), (6, 2))] + \
        [("u8", (19, 14), 1, rc, 2) for rc in (3, 4, 5, 6, 7)] + \
        [("u16", g, 2, 3, rf) for g in ((29, 15), (14, 3), (3, 29)) for rf in (1, 2)]


@pytest.mark.parametrize("dtype,grid,levels,rc,rf", CASES)
def test_predict_parents_over_row_ends(dtype, grid, levels, rc, rf):
    from paper_2504_17987_amd import api
    u16 = dtype == "u16"
    step = 12 if u16 else 8
    W, H, n = step * grid[0], step * grid[1], 2
    prs = []
    for k in range(n):
        flow = synth.LambOseen.with_peak(W / 2.0, H / 2.0, max(min(W, H) / 4.0, 4.0), rc * 2 ** (levels - 1), 1 - 2 * k)
        prs.append(synth.make_pair(W, H, flow, 0.05, noise=32.0 if u16 else 2.0, seed=70 + k, maxval=65535 if u16 else 255,
                                   I0=(30000.0, 65535.0) if u16 else (120.0, 255.0), dtype=np.uint16 if u16 else np.uint8))

    def dev(x):
        t = torch.from_numpy(np.ascontiguousarray(x).view(np.int16) if u16 else np.ascontiguousarray(x)).cuda()
        return t.view(torch.uint16) if u16 else t
    P = api.Plan(W, H, max_batch=n, win=2 * step, step=step, levels=levels, radius_coarse=rc, radius_fine=rf, dtype=dtype,
                 bit_depth=16 if u16 else None)
    got = P.predict(dev(np.stack([p[0] for p in prs])), dev(np.stack([p[1] for p in prs]))).cpu().numpy()
    for i, (a, b) in enumerate(prs):
        ref = oracle.predict(a, b, step, 2 * step, levels, rc, rf).astype(np.float32)
        assert np.array_equal(got[i], ref), (i, np.argwhere(got[i] != ref)[:4])


@pytest.mark.parametrize("rf", [1, 2])
def test_predict_many_pairs_as_few(rf):
    from paper_2504_17987_amd import api
    W, H, n = 8 * 43, 8 * 27, 20
    rng = np.random.default_rng(rf)
    A = rng.integers(0, 256, (2, H, W), dtype=np.uint8)
    B = np.where(rng.random((2, H, W)) < 0.3, rng.integers(0, 256, (2, H, W), dtype=np.uint8), np.roll(A, (3, -5), (1, 2)))
    ref = [oracle.predict(A[i], B[i], 8, 16, 2, 6, rf).astype(np.float32) for i in range(2)]
    P = api.Plan(W, H, max_batch=n, levels=2, radius_coarse=6, radius_fine=rf)
    rep = lambda x: torch.from_numpy(np.ascontiguousarray(np.tile(x, (n // 2, 1, 1)))).cuda()  # noqa: E731
    got = P.predict(rep(A), rep(B)).cpu().numpy()
    for i in range(n):
        assert np.array_equal(got[i], ref[i % 2]), i
