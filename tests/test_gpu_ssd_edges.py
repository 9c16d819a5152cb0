"""Windowed SSD and its adjoint at the edges of the tiled kernels: grids of
two to a few nodes, a last tile one or two nodes wide, samples that leave the
frame by a column or by far, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import TOL_REL, say
from test_gpu_ssd import cell_edge_nodes, dev, f32_pairs

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("W,H,amp", [(16, 16, 3.0), (24, 136, 9.0), (144, 80, 2.0), (80, 144, 40.0), (200, 72, 300.0)])
def test_ssd_tiles_at_frame_edges(W, H, amp):
    from paper_2504_17987_amd import api
    say(f"[ssd edges] {W}x{H} up to {amp} px")
    A, B, T = f32_pairs(2, W, H)
    rng = np.random.default_rng(int(W * 1000 + H))
    U = rng.uniform(-amp, amp, T.shape).astype(np.float32)
    g = rng.uniform(0.5, 1.5, (2,) + T.shape[2:]).astype(np.float32)
    g[1, 0, 0] = 0.0
    P = api.Plan(W, H, max_batch=2, dtype="f32", levels=1, win=16, step=8)
    loss = P.ssd_forward(dev(A), dev(B), dev(U)).cpu().numpy()
    gU, D = (x.cpu().numpy() for x in P.ssd_backward(dev(A), dev(B), dev(U), dev(g)))
    for i in range(2):
        Ai, Bi, Ui = A[i].astype(np.float64), B[i].astype(np.float64), U[i].astype(np.float64)
        lo = oracle.ssd_forward(Ai, Bi, Ui, 16, 8)
        go, Do = oracle.ssd_grad(Ai, Bi, Ui, g[i].astype(np.float64), 16, 8)
        # FP32 positions of up to `amp` px next to FP64 ones: half an ulp of the position times the slope
        tol = TOL_REL * max(1.0, amp / 8.0)
        assert np.abs(loss[i] - lo).max() <= tol * np.abs(lo).max()
        ok = ~cell_edge_nodes(Ui, W, H, eps=1e-4 * max(1.0, amp / 8.0))
        assert np.abs(gU[i] - go)[ok].max(initial=0) <= tol * max(np.abs(go).max(), 1e-30)
        assert np.abs(D[i] - Do)[ok].max(initial=0) <= tol * max(np.abs(Do).max(), 1e-30)


def test_ssd_nan_and_huge_nodes_stay_local():
    """A NaN node spoils the windows whose pixels interpolate it and no other;
    nodes far beyond 32-bit positions leave every sample outside, zero."""
    from paper_2504_17987_amd import api
    A, B, T = f32_pairs(2, 136, 104)
    U = T.astype(np.float32)
    U[0, :, 6, 7] = np.nan
    U[1] = 1e30
    P = api.Plan(136, 104, max_batch=2, dtype="f32", levels=1, win=16, step=8)
    loss = P.ssd_forward(dev(A), dev(B), dev(U)).cpu().numpy()
    clean = P.ssd_forward(dev(A), dev(B), dev(T.astype(np.float32))).cpu().numpy()
    bad = np.zeros(clean[0].shape, bool)
    bad[5:8, 6:9] = True
    assert np.isnan(loss[0][bad]).all() and np.array_equal(loss[0][~bad] == clean[0][~bad], np.ones((~bad).sum(), bool))
    pad = np.pad(A[1].astype(np.float64) ** 2, 4)
    want = np.array([[pad[8 * i:8 * i + 16, 8 * j:8 * j + 16].sum() for j in range(17)] for i in range(13)])
    assert np.isfinite(loss[1]).all()
    np.testing.assert_allclose(loss[1], want, rtol=TOL_REL)
