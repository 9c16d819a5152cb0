"""A predictor node that is not finite spoils the windows that its
interpolation reaches (three nodes off it reaches none) and no others,
wherever it lies in a kernel's tile of windows."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import compare_correct, say
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("W,H,win,dtype,r,warp", [
    (560, 528, 32, "u8", 4, "b"), (560, 528, 32, "u8", 4, "central"), (400, 304, 32, "u16", 8, "b"),
    (400, 304, 32, "u16", 8, "central"), (720, 688, 32, "u8", 1, "central"), (208, 176, 32, "u8", 4, "central"),
    (264, 200, 16, "u8", 4, "b"), (264, 200, 16, "u8", 4, "central"), (264, 200, 16, "u16", 4, "central"),
    (264, 200, 16, "u16", 1, "b"), (300, 228, 24, "u16", 4, "b")])
def test_one_node_not_finite(W, H, win, dtype, r, warp, value):
    from paper_2504_17987_amd import api
    say(f"[node {value}] {W}x{H} win {win} {dtype} r {r} {warp}")
    step, u16, mode = win // 2, dtype == "u16", int(warp == "central")
    flow = synth.LambOseen.with_peak((W - 1) / 2, (H - 1) / 2, min(W, H) / 5, 2.5 if r > 1 else 0.8)
    A, B = synth.make_pair(W, H, flow, 0.04, noise=32.0 if u16 else 2.0, I0=(1920.0, 4095.0) if u16 else (120.0, 255.0),
                           dtype=np.uint16 if u16 else np.uint8, maxval=4095 if u16 else 255, seed=31)
    pred = (np.round(2 * synth.truth(flow, W, H, step)) / 2).astype(np.float32)
    P = api.Plan(W, H, win=win, step=step, radius=max(r, 4), levels=1, radius_coarse=4, dtype=dtype, warp=warp,
                 peak="fixed" if r == 1 else "argmax")
    do, po, fo = oracle.correct(A, B, win, step, max(r, 4), pred.astype(np.float64), mode, int(r == 1))
    dev = [(torch.from_numpy(x[None].view(np.int16)).view(torch.uint16) if u16 else torch.from_numpy(x[None])).cuda()
           for x in (A, B)]
    for na, nb in ((8, 8), (6, 8), (12, 16)):   # corners of the kernels' tiles (4 x 4, 4 x 2 and 8 x 6 windows)
        if na >= P.ny or nb >= P.nx:
            continue
        p1 = pred.copy()
        p1[:, na, nb] = value
        d, p, f = (x.cpu().numpy()[0] for x in P.correct(*dev, torch.from_numpy(p1[None]).cuda()))
        far = np.maximum(np.abs(np.arange(P.ny) - na)[:, None], np.abs(np.arange(P.nx) - nb)[None, :]) >= 3
        d, p, f = np.where(far, d, do), np.where(far, p, po), np.where(far, f, fo)
        compare_correct(None, None, A.astype(float), B.astype(float), win, step, max(r, 4), pred.astype(np.float64), d, p,
                        f, do, po, fo, mode=mode, fixed=r == 1, where=f"node ({na},{nb}) not finite, win {win} {warp}")
