"""Correlation of 32 px windows at 50% overlap (k_correct_rows) against the
FP64 oracle: both tilings (a workgroup per window, a shared tile), every
radius it is built for, u8 and u16 frames, both deformations, grids that end
inside a tile, grids of one node, predictors too steep for the staged box and
padded rows.  Tolerances as for the other correlation kernels: 0.01 px, 2e-5
in the coefficient, flags equal, explained exemptions only."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import compare_correct, say
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# name: (W, H, dtype, radius, peak, warp, predictor, row padding in px)
CASES = {
    "window_r4": (256, 208, "u8", 4, "argmax", "b", "flow", 0),
    "window_r4_nopred": (256, 208, "u8", 4, "argmax", "b", None, 0),
    "window_r4_central_u16": (176, 144, "u16", 4, "argmax", "central", "flow", 6),
    "window_r8_u16": (208, 176, "u16", 8, "argmax", "b", "flow", 0),
    "window_r8_central": (208, 176, "u8", 8, "argmax", "central", "flow", 0),
    "window_fixed": (256, 208, "u8", 8, "fixed", "b", "flow", 0),
    "window_fixed_central_u16": (256, 208, "u16", 4, "fixed", "central", "flow", 0),
    "window_r8_steep": (208, 176, "u8", 8, "argmax", "b", "steep", 0),
    "one_node": (16, 16, "u8", 4, "argmax", "b", "flow", 0),
    "one_column_r8": (16, 160, "u8", 8, "argmax", "central", "flow", 0),
    "tile_r4": (592, 528, "u8", 4, "argmax", "b", "flow", 4),
    "tile_r4_steep": (560, 528, "u8", 4, "argmax", "b", "steep", 0),
    "tile_r4_central": (560, 528, "u8", 4, "argmax", "central", "flow", 0),
    "tile_r4_u16": (560, 528, "u16", 4, "argmax", "b", "flow", 2),
    "tile_r4_central_u16": (592, 528, "u16", 4, "argmax", "central", "steep", 0),
    "tile_r8": (368, 304, "u8", 8, "argmax", "b", "flow", 0),
    "tile_r8_u16_nopred": (400, 272, "u16", 8, "argmax", "b", None, 0),
    "tile_r8_central": (368, 304, "u8", 8, "argmax", "central", "steep", 0),
    "tile_fixed": (720, 688, "u8", 4, "fixed", "b", "flow", 0),
    "tile_fixed_central_u16": (688, 640, "u16", 4, "fixed", "central", "flow", 0),
}


@pytest.mark.parametrize("case", list(CASES))
def test_correct_32px_windows(case):
    from paper_2504_17987_amd import api
    say(f"[correct 32 px] {case}")
    W, H, dtype, r, peak, warp, pk, pad = CASES[case]
    flow = synth.LambOseen.with_peak((W - 1) / 2, (H - 1) / 2, min(W, H) / 5, 2.5 if peak == "argmax" else 0.8)
    u16 = dtype == "u16"
    A, B = synth.make_pair(W, H, flow, 0.03, noise=32.0 if u16 else 2.0, I0=(1920.0, 4095.0) if u16 else (120.0, 255.0),
                           dtype=np.uint16 if u16 else np.uint8, maxval=4095 if u16 else 255, seed=11)
    pred = None
    if pk == "flow":
        pred = np.round(2 * synth.truth(flow, W, H, 16)) / 2
    elif pk == "steep":   # a spread of more than 17 px across a tile; the windows still match in places
        pred = synth.truth(flow, W, H, 16)
        pred[0] += 0.4 * ((np.arange(W // 16) * 16)[None, :] - W / 2)
    if pred is not None:
        pred = pred.astype(np.float32).astype(np.float64)
    mode, fixed = int(warp == "central"), peak == "fixed"
    do, po, fo = oracle.correct(A, B, 32, 16, r, pred, mode, int(fixed))
    P = api.Plan(W, H, win=32, step=16, radius=r, levels=1, radius_coarse=4, dtype=dtype, peak=peak, warp=warp)
    assert P.correct_impl() == 1

    def dev(x):
        rows = np.full((1, H, W + pad), x.max(), x.dtype)   # what lies in the padding is never read as a pixel
        rows[0, :, :W] = x
        t = torch.from_numpy(rows.view(np.int16) if u16 else rows).cuda()
        return (t.view(torch.uint16) if u16 else t)[:, :, :W]
    pg = None if pred is None else torch.from_numpy(pred[None].astype(np.float32)).cuda()
    d, p, f = (x.cpu().numpy()[0] for x in P.correct(dev(A), dev(B), pg))
    compare_correct(None, None, A.astype(float), B.astype(float), 32, 16, r, pred, d, p, f, do, po, fo, mode=mode,
                    fixed=fixed, where=f"correct 32 px [{case}]")


def test_batch_does_not_change_a_pair():
    """Bitwise: a pair alone and in a batch large enough for any tiling."""
    from paper_2504_17987_amd import api
    W, H, n = 256, 256, 8
    prs = [synth.make_pair(W, H, synth.Uniform(1.3 + 0.2 * i, -0.7), 0.03, seed=i) for i in range(n)]
    A, B = (torch.from_numpy(np.stack([q[k] for q in prs])).cuda() for k in range(2))
    P = api.Plan(W, H, max_batch=n, win=32, step=16, radius=4, levels=1, radius_coarse=4)
    pred = torch.full((n, 2, 16, 16), 1.0, device="cuda")
    every = P.correct(A, B, pred)
    for i in range(n):
        one = P.correct(A[i:i + 1], B[i:i + 1], pred[i:i + 1])
        assert all(torch.equal(x[i], y[0]) for x, y in zip(every, one)), i
