"""Correlation under uneven light: the mean level differs from window to
window by many times the particles' contrast.  Sums taken about a level that
is not the window's own lose bits there, so the coefficient is held to a
tighter bound than elsewhere: about the window's own mean its sums have terms
of the size of the result, and FP32 chains of at most 256 such terms (the
errors of half of them cancelling) stay below 64 x 2^-24 = 4e-6."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import compare_correct, say
from paper_2504_17987_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

OWN_MEAN = 64 * 2.0 ** -24


def _dev(x):
    return (torch.from_numpy(x[None].copy()) if x.dtype == np.uint8
            else torch.from_numpy(x[None].view(np.int16).copy()).view(torch.uint16)).cuda()


def _lit_pair(W, H, u16, level, swing, contrast, peak):
    """Particles of `contrast` grey levels under light of `level` +- `swing`."""
    flow = synth.LambOseen.with_peak((W - 1) / 2, (H - 1) / 2, min(W, H) / 5, peak)
    pair = synth.make_pair(W, H, flow, 0.04, noise=0.0, I0=(2000.0, 4000.0), dtype=np.uint16, maxval=4095, seed=5)
    rng = np.random.default_rng(9)
    y, x = np.mgrid[:H, :W]
    light = level + swing * np.sin(x * (2 * np.pi / 170)) * np.cos(y * (2 * np.pi / 150))
    out = [np.clip(np.rint(light + I * (contrast / 3000.0) + 0.02 * contrast * rng.standard_normal(I.shape)), 0,
                   4095 if u16 else 255).astype(np.uint16 if u16 else np.uint8) for I in pair]
    return out, flow


# name: (W, H, win, dtype, radius, peak, warp)
LIGHT = {
    "window_r4": (256, 208, 32, "u8", 4, "argmax", "b"),
    "window_r8_central_u16": (208, 176, 32, "u16", 8, "argmax", "central"),
    "tile_r4": (560, 528, 32, "u8", 4, "argmax", "b"),
    "tile_r4_u16": (560, 528, 32, "u16", 4, "argmax", "b"),
    "tile_r4_central": (560, 528, 32, "u8", 4, "argmax", "central"),
    "tile_r4_central_u16": (560, 528, 32, "u16", 4, "argmax", "central"),
    "tile_r8_u16": (400, 304, 32, "u16", 8, "argmax", "b"),
    "tile_r8_central_u16": (400, 304, 32, "u16", 8, "argmax", "central"),
    "tile_fixed_u16": (720, 688, 32, "u16", 4, "fixed", "b"),
}


@pytest.mark.parametrize("case", list(LIGHT))
def test_uneven_light(case):
    from paper_2504_17987_amd import api
    say(f"[uneven light] {case}")
    W, H, win, dtype, r, peak, warp = LIGHT[case]
    u16, fixed, mode, step = dtype == "u16", peak == "fixed", int(warp == "central"), win // 2
    (A, B), flow = _lit_pair(W, H, u16, *((3000, 600, 300) if u16 else (100, 80, 15)), 0.8 if fixed else 2.5)
    pred = (np.round(2 * synth.truth(flow, W, H, step)) / 2).astype(np.float32)
    do, po, fo = oracle.correct(A, B, win, step, r, pred.astype(np.float64), mode, int(fixed))
    P = api.Plan(W, H, win=win, step=step, radius=r, levels=1, radius_coarse=4, dtype=dtype, peak=peak, warp=warp)
    d, p, f = (x.cpu().numpy()[0] for x in P.correct(_dev(A), _dev(B), torch.from_numpy(pred[None]).cuda()))
    ex = compare_correct(None, None, A.astype(float), B.astype(float), win, step, r, pred.astype(np.float64), d, p, f,
                         do, po, fo, mode=mode, fixed=fixed, where=f"uneven light [{case}]")
    assert np.abs(p - po)[~ex].max() < OWN_MEAN


@pytest.mark.parametrize("W,H", [(256, 208), (560, 528)])   # a workgroup per window, a shared tile
@pytest.mark.parametrize("dtype,level,up", [("u8", 100, 32), ("u16", 1000, 2000)])
@pytest.mark.parametrize("warp", ["b", "central"])
def test_nearly_constant_window_off_its_surroundings(W, H, dtype, level, up, warp):
    """A 32 px window that is constant but for one pixel is not flat, however
    far its level is from that of the windows around it."""
    from paper_2504_17987_amd import api
    say(f"[nearly constant window] {W}x{H} {dtype} {warp}")
    rng = np.random.default_rng(3)
    A = rng.integers(level - 20, level + 21, (H, W)).astype(np.uint16 if dtype == "u16" else np.uint8)
    nodes = [(a, b) for a in range(2, H // 16 - 3, 5) for b in range(2, W // 16 - 3, 5)]
    for a, b in nodes:   # window (a, b): rows 16 a - 8 .. 16 a + 23; 4 px more for the shifts
        y, x = 16 * a - 8, 16 * b - 8
        A[y - 4:y + 36, x - 4:x + 36] = level + up
        A[y + 13 + a % 4, x + 14 + b % 4] += 1
    P = api.Plan(W, H, win=32, step=16, radius=4, levels=1, radius_coarse=4, dtype=dtype, warp=warp)
    zero = torch.zeros((1, 2, P.ny, P.nx), device="cuda")
    d, p, f = (x.cpu().numpy()[0] for x in P.correct(_dev(A), _dev(A), zero))
    do, po, fo = oracle.correct(A, A, 32, 16, 4, np.zeros((2, P.ny, P.nx)), int(warp == "central"), 0)
    for a, b in nodes:
        assert fo[a, b] == 0 and po[a, b] == pytest.approx(1.0)
        assert f[a, b] == 0 and abs(p[a, b] - 1.0) < OWN_MEAN and np.abs(d[:, a, b] - do[:, a, b]).max() < 0.01, (
            a, b, f[a, b], p[a, b], d[:, a, b])


@pytest.mark.parametrize("W,H", [(264, 200), (520, 400)])
@pytest.mark.parametrize("dtype,light", [("u8", (200, 10, 25)), ("u16", (3000, 100, 300))])
def test_bright_frames_both_deformed_16px(W, H, dtype, light):
    """16 px windows with both frames deformed: bright frames whose level
    varies little over a tile of windows, on grids that end inside a tile.
    (The sums run about the tile's mean, and the light's swing is at most
    twice the particles' standard deviation: terms at most 4 or 5 times the
    result's size, within the usual 2e-5.)"""
    from paper_2504_17987_amd import api
    say(f"[bright frames, 16 px, both deformed] {W}x{H} {dtype}")
    (A, B), flow = _lit_pair(W, H, dtype == "u16", *light, 2.5)
    pred = (np.round(2 * synth.truth(flow, W, H, 8)) / 2).astype(np.float32)
    do, po, fo = oracle.correct(A, B, 16, 8, 4, pred.astype(np.float64), 1, 0)
    P = api.Plan(W, H, win=16, step=8, radius=4, levels=1, radius_coarse=4, dtype=dtype, warp="central")
    d, p, f = (x.cpu().numpy()[0] for x in P.correct(_dev(A), _dev(B), torch.from_numpy(pred[None]).cuda()))
    compare_correct(None, None, A.astype(float), B.astype(float), 16, 8, 4, pred.astype(np.float64), d, p, f, do, po, fo,
                    mode=1, where=f"bright frames [{W}x{H} {dtype}]")
