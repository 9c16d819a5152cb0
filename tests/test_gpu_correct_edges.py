"""Correlation by two waves per shift band (k_correct_halves) against the FP64
oracle: 24 px u16 windows with frame B deformed and 16 px windows with both
deformed, on grids that end inside a tile (8 x 6 windows), of one node, with
predictors too steep for the staged box, far beyond it, none, and padded
rows.  Tolerances as for the other correlation kernels."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import compare_correct, say
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# name: (W, H, dtype, win, warp, predictor, row padding in px)
CASES = {
    "u16_24": (396, 228, "u16", 24, "b", "flow", 0),
    "u16_24_tile": (96, 72, "u16", 24, "b", "flow", 6),
    "u16_24_nopred": (204, 156, "u16", 24, "b", None, 2),
    "u16_24_steep": (300, 228, "u16", 24, "b", "steep", 0),
    "u16_24_far": (204, 156, "u16", 24, "b", "far", 0),
    "u16_24_one_node": (12, 12, "u16", 24, "b", "flow", 0),
    "u16_24_row": (132, 12, "u16", 24, "b", "flow", 0),
    "u8_central": (264, 200, "u8", 16, "central", "flow", 4),
    "u8_central_tile": (64, 48, "u8", 16, "central", "flow", 0),
    "u8_central_nopred": (136, 104, "u8", 16, "central", None, 0),
    "u8_central_steep": (200, 152, "u8", 16, "central", "steep", 0),
    "u8_central_far": (136, 104, "u8", 16, "central", "far", 0),
    "u8_central_one_node": (8, 8, "u8", 16, "central", "flow", 0),
    "u16_central": (200, 104, "u16", 16, "central", "flow", 2),
    "u16_central_steep": (200, 152, "u16", 16, "central", "steep", 0),
}


@pytest.mark.parametrize("case", list(CASES))
def test_correct_halves(case):
    from paper_2504_17987_amd import api
    say(f"[correct halves] {case}")
    W, H, dtype, win, warp, pk, pad = CASES[case]
    step = win // 2
    flow = synth.LambOseen.with_peak((W - 1) / 2, (H - 1) / 2, max(min(W, H) / 5, 4.0), 2.5)
    u16 = dtype == "u16"
    A, B = synth.make_pair(W, H, flow, 0.04, noise=32.0 if u16 else 2.0, I0=(1920.0, 4095.0) if u16 else (120.0, 255.0),
                           dtype=np.uint16 if u16 else np.uint8, maxval=4095 if u16 else 255, seed=21)
    pred = None
    if pk is not None:
        pred = np.round(2 * synth.truth(flow, W, H, step)) / 2
        if pk == "steep":   # a spread of more than 24 px across a tile
            pred[0] += 0.5 * ((np.arange(W // step) * step)[None, :] - W / 2)
        if pk == "far":     # beyond 100 px at some nodes only
            pred[1, :, : pred.shape[2] // 2] = 104.0
        pred = pred.astype(np.float32).astype(np.float64)
    mode = int(warp == "central")
    do, po, fo = oracle.correct(A, B, win, step, 4, pred, mode, 0)
    P = api.Plan(W, H, win=win, step=step, radius=4, levels=1, radius_coarse=4, dtype=dtype, warp=warp)

    def dev(x):
        rows = np.full((1, H, W + pad), x.max(), x.dtype)   # what lies in the padding is never read as a pixel
        rows[0, :, :W] = x
        t = torch.from_numpy(rows.view(np.int16) if u16 else rows).cuda()
        return (t.view(torch.uint16) if u16 else t)[:, :, :W]
    pg = None if pred is None else torch.from_numpy(pred[None].astype(np.float32)).cuda()
    d, p, f = (x.cpu().numpy()[0] for x in P.correct(dev(A), dev(B), pg))
    compare_correct(None, None, A.astype(float), B.astype(float), win, step, 4, pred, d, p, f, do, po, fo, mode=mode,
                    where=f"correct halves [{case}]", max_flat=24 if pk in ("steep", "far") else 8)
