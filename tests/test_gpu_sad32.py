"""Block search of 32x32 blocks at step 16 (k_sad_coarse32, k_sad_fine32)
against the integer oracle, bit for bit: every radius they are built for, both
tilings of the coarsest level (few nodes, 4,096 and more), odd grids that end
inside a tile or a parent, one node, u8 and u16, and radii beyond them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# W, H, pairs, dtype, levels, radius_coarse, radius_fine
CASES = [(272, 208, 2, "u8", 1, r, 2) for r in range(2, 10)] + \
        [(272, 208, 2, "u16", 1, r, 2) for r in range(2, 10)] + \
        [(272, 208, 20, "u8", 1, r, 2) for r in (3, 4, 5, 6, 7, 8)] + \
        [(272, 208, 20, "u16", 1, r, 2) for r in (3, 6, 7, 8)] + \
        [(16, 16, 1, "u8", 1, 8, 2), (16, 16, 1, "u16", 2, 3, 2), (48, 16, 2, "u8", 3, 4, 2)] + \
        [(304, 240, 2, dt, lv, 4, rf) for dt in ("u8", "u16") for lv in (2, 3) for rf in (0, 1, 2, 3)]


@pytest.mark.parametrize("W,H,n,dtype,levels,rc,rf", CASES)
def test_predict_32px_blocks(W, H, n, dtype, levels, rc, rf):
    from paper_2504_17987_amd import api
    u16 = dtype == "u16"
    prs = []
    for k in range(min(n, 2)):
        flow = synth.LambOseen.with_peak(W / 2.0, H / 2.0, max(min(W, H) / 4.0, 4.0), min(rc * 2 ** (levels - 1), 20), 1 - 2 * k)
        prs.append(synth.make_pair(W, H, flow, 0.03, noise=32.0 if u16 else 2.0, seed=50 + k, maxval=65535 if u16 else 255,
                                   I0=(30000.0, 65535.0) if u16 else (120.0, 255.0), dtype=np.uint16 if u16 else np.uint8))
    A, B = (np.stack([prs[i % len(prs)][k] for i in range(n)]) for k in range(2))

    def dev(x):
        t = torch.from_numpy(x.view(np.int16) if u16 else x).cuda()
        return t.view(torch.uint16) if u16 else t
    P = api.Plan(W, H, max_batch=n, win=32, step=16, levels=levels, radius_coarse=rc, radius_fine=rf, dtype=dtype,
                 bit_depth=16 if u16 else None)
    got = P.predict(dev(A), dev(B)).cpu().numpy()
    for i in range(n):
        a, b = prs[i % len(prs)]
        if i < len(prs):
            ref = oracle.predict(a, b, 16, 32, levels, rc, rf).astype(np.float32)
            assert np.array_equal(got[i], ref), (i, np.argwhere(got[i] != ref)[:4])
        else:
            assert np.array_equal(got[i], got[i % len(prs)]), i
