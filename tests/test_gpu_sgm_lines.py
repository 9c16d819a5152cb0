"""Semi-global matching where a line's two paths meet: lines of one, two, odd
and even numbers of nodes, for every number of candidates per lane, against
the integer oracle, bit for bit; repeated, since the paths run side by side."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("nx,ny", [(2, 1), (1, 2), (1, 7), (2, 2), (3, 4), (9, 5), (16, 33)])
@pytest.mark.parametrize("rc", [3, 6, 8, 12])
def test_sgm_lines_meet_in_the_middle(nx, ny, rc):
    from paper_2504_17987_amd import api
    W, H, n = max(8 * nx, 16), max(8 * ny, 16), 3
    rng = np.random.default_rng(nx * 100 + ny + rc)
    A = rng.integers(0, 256, (n, H, W), dtype=np.uint8)
    B = np.where(rng.random((n, H, W)) < 0.5, np.roll(A, (2, -3), (1, 2)), rng.integers(0, 256, (n, H, W), dtype=np.uint8))
    P = api.Plan(W, H, max_batch=n, levels=1, radius_coarse=rc, sgm=True)
    a, b = torch.from_numpy(A).cuda(), torch.from_numpy(np.ascontiguousarray(B)).cuda()
    ref = np.stack([oracle.predict(A[i], B[i], 8, 16, 1, rc, 2, True, (2, 16)) for i in range(n)]).astype(np.float32)
    for _ in range(4):
        assert np.array_equal(P.predict(a, b).cpu().numpy(), ref)
