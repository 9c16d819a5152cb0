"""The work that this framework is timed on: its public entry points over the
range of sizes, data types and options that its users run.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare(case, seed)`` makes what a user's program holds before the call (the
frames on the GPU, the plan with its workspace, the output tensors),
``run(state)`` is one pass through the public API, ``work(case)`` what a pass
cannot do without, and ``exact(case, seed)`` the same outputs in 64 bits from
plain torch.

Kinds of case:
  run         Plan.run: the whole path, frames in, validated field and vorticity out
  predict     Plan.predict: the coarse-to-fine block search alone
  correct     Plan.correct: deformation, correlation and fit about a given predictor
  ssd         autograd.warp_ssd forward and its gradient (float32 frames)
  preprocess  Plan.highpass then Plan.clahe
"""
import math

import torch

from paper_2504_17987_amd import api, autograd

# Defaults of a case: the processing parameters of a 1 MP u8 pair.
_BASE = dict(dtype="u8", n=1, win=16, radius=4, levels=3, rc=6, rf=2, warp="b", peak="argmax", sgm=False,
             flow="vortex", ppp=0.04, dropout=0.1)


def _case(name, kind, w, h, **kw):
    c = dict(_BASE, kind=kind, w=w, h=h)
    c.update(kw)
    if kind in ("ssd", "preprocess"):
        c = {k: c[k] for k in c if k in ("kind", "w", "h", "n", "dtype", "ppp", "dropout", "flow",
                                      "levels", "rc", "rf", "hp_radius", "tiles_x", "tiles_y", "clip")}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the headline workload: a recorded sequence of 1 MP frames in batches of 64 pairs
        _case("run_1mp_u8_b64", "run", 1024, 1024, n=64),
        # live display: one camera pair at a time, where latency and launches count
        _case("run_1mp_u8_b1", "run", 1024, 1024),
        # the largest frames, one pair
        _case("run_8192x4096_u8_b1", "run", 8192, 4096),
        # the smallest call: a 256^2 region of interest, 32 px windows, +-8 px
        _case("run_256_u8_win32_r8", "run", 256, 256, win=32, radius=8, levels=1, rc=8, flow="uniform", ppp=0.03,
              dropout=0.0),
        # a sparsely seeded wake behind a cylinder: 32 px windows, few particles
        _case("run_wake_u8_win32_b4", "run", 1024, 512, n=4, win=32, levels=2, flow="wake", ppp=0.002, dropout=0.0),
        # a 4K 12-bit camera, batches of 8 pairs: the predictor, and the correlation about it
        _case("predict_4k_u16_b8", "predict", 3840, 2160, n=8, dtype="u16", win=24, ppp=0.02, dropout=0.0),
        _case("correct_4k_u16_b8", "correct", 3840, 2160, n=8, dtype="u16", win=24, ppp=0.02, dropout=0.0),
        # the symmetric deformation of both frames, on a ragged frame size
        _case("correct_1000x760_central_b16", "correct", 1000, 760, n=16, warp="central"),
        # the semi-global predictor on the headline frames
        _case("predict_1mp_sgm_b64", "predict", 1024, 1024, n=64, sgm=True),
        # differentiable refinement: the windowed SSD and its gradient
        _case("ssd_512_b64", "ssd", 512, 512, n=64, dtype="f32", ppp=0.05),
        # background removal and contrast equalisation of 64 frames
        _case("preprocess_1mp_u8_b64", "preprocess", 1024, 1024, n=64, hp_radius=7, tiles_x=8, tiles_y=8, clip=2.0),
        # the same of 4K 12-bit frames, tiles that do not divide the frame
        _case("preprocess_4k_u16_b8", "preprocess", 3840, 2160, n=8, dtype="u16", ppp=0.02, hp_radius=5, tiles_x=7,
              tiles_y=5, clip=3.0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, step, lo, hi):
    """A side of lo..hi px, a multiple of the vector spacing."""
    return max(lo, step * int(round(_logint(rng, lo, hi) / step)))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "predict", "correct", "correct", "ssd", "preprocess"])
    if kind == "ssd":
        w, h = _size(rng, 8, 128, 1024), _size(rng, 8, 128, 1024)
        return _case("", kind, w, h, n=_logint(rng, 1, max(1, min(64, (1 << 24) // (w * h)))), dtype="f32", ppp=0.05)
    if kind == "preprocess":
        dt = rng.choice(["u8", "u16"])
        w, h = _size(rng, 8, 256, 4096), _size(rng, 8, 256, 2304)
        return _case("", kind, w, h, n=_logint(rng, 1, max(1, min(64, (1 << 25) // (w * h)))), dtype=dt,
                     ppp=rng.choice([0.02, 0.04]), hp_radius=rng.randint(3, 15), tiles_x=rng.randint(4, 16),
                     tiles_y=rng.randint(4, 16), clip=rng.choice([1.5, 2.0, 3.0, 4.0]))
    geo = rng.choice(["16", "16", "24", "32"])
    warp = rng.choice(["b", "b", "b", "central"])
    if geo == "16":
        dt = rng.choice(["u8", "u8", "u16"])
        w, h = _size(rng, 8, 256, 4096), _size(rng, 8, 256, 4096)
        most = (1 << 25) if warp == "b" and dt == "u8" else 1 << 23
        return _case("", kind, w, h, n=_logint(rng, 1, max(1, min(64, most // (w * h)))), dtype=dt, warp=warp,
                     rc=rng.randint(4, 7), peak=rng.choice(["argmax", "argmax", "fixed"]),
                     sgm=rng.random() < 0.2 and dt == "u8", ppp=rng.choice([0.03, 0.04]))
    if geo == "24":
        w, h = _size(rng, 12, 384, 3840), _size(rng, 12, 384, 2160)
        most = (1 << 25) if warp == "b" else 1 << 23
        return _case("", kind, w, h, n=_logint(rng, 1, max(1, min(8, most // (w * h)))), dtype="u16", win=24,
                     warp=warp, rc=rng.randint(4, 7), ppp=0.02, dropout=rng.choice([0.0, 0.1]))
    w, h = _size(rng, 16, 256, 2048), _size(rng, 16, 256, 2048)
    r = rng.choice([4, 4, 8])
    return _case("", kind, w, h, n=_logint(rng, 1, max(1, min(16, ((1 << 22) if r == 4 else (1 << 21)) // (w * h)))),
                 dtype=rng.choice(["u8", "u8", "u16"]), win=32, radius=r, levels=rng.choice([1, 2, 3]),
                 rc=rng.choice([6, 8]), warp=warp, peak=rng.choice(["argmax", "argmax", "fixed"]),
                 flow=rng.choice(["wake", "vortex"]), ppp=rng.choice([0.005, 0.02]))


# ---------------------------------------------------------------------------
# inputs: seeded particle images of an analytic flow
# ---------------------------------------------------------------------------

def _step(c):
    return 8 if c["kind"] in ("ssd", "preprocess") else c["win"] // 2


def _reach(c):
    """Largest displacement that the predictor of the case can find (px)."""
    s = 1 << (c["levels"] - 1)
    return c["rc"] * s + c["rf"] * (s - 1)


def _vortex(x, y, xc, yc, rc, peak):
    """Lamb-Oseen vortex of the given core radius and peak displacement."""
    dx, dy = x - xc, y - yc
    r2 = (dx * dx + dy * dy).clamp_min(1e-9)
    k = peak / 0.638161 * rc * -torch.expm1(-r2 / rc ** 2) / r2
    return -k * dy, k * dx


def _flow(c, gen):
    """(x, y) -> (u, v), px per frame pair."""
    w, h = float(c["w"]), float(c["h"])
    j = torch.rand(4, generator=gen, device="cuda", dtype=torch.float64).tolist()
    if c["kind"] == "ssd":   # smooth random flow of at most 6 px: a few modes
        m = torch.rand((8, 6), generator=gen, device="cuda", dtype=torch.float64)

        def smooth(x, y):
            u, v = torch.zeros_like(x), torch.zeros_like(x)
            for k in range(8):
                kx, ky = (m[k, 0] - 0.5) / 8, (m[k, 1] - 0.5) / 8
                ph = kx * x + ky * y + 6.283 * m[k, 2]
                u = u + 0.75 * (2 * m[k, 3] - 1) * torch.sin(ph)
                v = v + 0.75 * (2 * m[k, 4] - 1) * torch.sin(ph + m[k, 5])
            return u, v
        return smooth
    if c["flow"] == "uniform":
        return lambda x, y: (torch.full_like(x, 3.4 + 0.6 * (j[0] - 0.5)), torch.full_like(x, -1.7 + 0.6 * (j[1] - 0.5)))
    if c["flow"] == "wake":   # free stream, deficit behind the body, staggered vortex street
        big = min(6.0, 0.5 * _reach(c))

        def wake(x, y):
            u = big - 0.5 * big * 0.5 * (1 + torch.tanh((x - w / 6) / (h / 8))) * torch.exp(-((y - h / 2) / (0.09 * h)) ** 2)
            v = torch.zeros_like(x)
            xk, k = w / 6 + (0.15 + 0.05 * j[0]) * h, 0
            while xk < w + h / 4:
                s = 1.0 if k % 2 == 0 else -1.0
                a, b = _vortex(x, y, xk, h / 2 + s * 0.075 * h, h / 16, -s * 0.4 * big)
                u, v = u + a, v + b
                xk, k = xk + h / 4, k + 1
            return u, v
        return wake
    rc, peak = min(w, h) / 8, min(20.0, 0.65 * _reach(c))
    xc, yc = w * (0.4 + 0.2 * j[0]), h * (0.4 + 0.2 * j[1])
    return lambda x, y: _vortex(x, y, xc, yc, rc, peak)


def _render(w, h, x, y, amp):
    """Pixel-integrated Gaussian particles of 2.5 px diameter.  Summed in
    fixed point, so that the order of the adds does not matter."""
    k = math.sqrt(8.0) / 2.5
    c = math.sqrt(math.pi) / (2 * k)
    img = torch.zeros(w * h + 1, dtype=torch.int64, device="cuda")
    off = torch.arange(-3, 4, device="cuda")
    for lo in range(0, x.numel(), 1 << 19):
        xs, ys, a = x[lo:lo + (1 << 19), None], y[lo:lo + (1 << 19), None], amp[lo:lo + (1 << 19), None, None]
        ix, iy = torch.floor(xs).long() + off, torch.floor(ys).long() + off
        ex = c * (torch.erf(k * (ix + 0.5 - xs)) - torch.erf(k * (ix - 0.5 - xs)))
        ey = c * (torch.erf(k * (iy + 0.5 - ys)) - torch.erf(k * (iy - 0.5 - ys)))
        val = torch.round(a * ey[:, :, None] * ex[:, None, :] * 65536.0).long()
        ok = ((ix >= 0) & (ix < w))[:, None, :] & ((iy >= 0) & (iy < h))[:, :, None]
        at = torch.where(ok, iy[:, :, None] * w + ix[:, None, :], w * h)
        img.scatter_add_(0, at.reshape(-1), val.reshape(-1))
    return img[:-1].reshape(h, w).double() / 65536.0


def _frames(c, seed):
    """(A, B) [n][h][w] of the case's type and the flow of each pair."""
    w, h, n = c["w"], c["h"], c["n"]
    top, noise, amp0, amp1 = (4095, 32.0, 1920.0, 4095.0) if c["dtype"] == "u16" else (255, 2.0, 120.0, 255.0)
    tdt = {"u8": torch.uint8, "u16": torch.uint16, "f32": torch.float32}[c["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(1000 + seed)
    A, B = (torch.empty((n, h, w), dtype=tdt, device="cuda") for _ in range(2))
    flows = []
    rand = lambda m: torch.rand(m, generator=gen, device="cuda", dtype=torch.float64)  # noqa: E731
    for i in range(n):
        flow = _flow(c, gen)
        flows.append(flow)
        m = int(c["ppp"] * (w + 32) * (h + 32))
        x, y, amp = rand(m) * (w + 32) - 16, rand(m) * (h + 32) - 16, amp0 + (amp1 - amp0) * rand(m)
        u, v = flow(x, y)
        keep = torch.where(rand(m) >= c.get("dropout", 0.0), amp, 0.0)
        for out, s, a in ((A, -0.5, amp), (B, 0.5, keep)):
            img = _render(w, h, x + s * u, y + s * v, a)
            img = img + noise * torch.randn((h, w), generator=gen, device="cuda", dtype=torch.float64)
            img = img.round().clamp(0, top)
            out[i] = (img / 255.0).float() if c["dtype"] == "f32" else img.int().to(tdt)
    return A, B, flows


def _nodes(c, flows, seed, err):
    """The flows at the vector nodes [n][2][ny][nx], float64; `err` px of noise."""
    s = _step(c)
    xs = torch.arange(c["w"] // s, device="cuda", dtype=torch.float64) * s + (s - 1) / 2
    ys = torch.arange(c["h"] // s, device="cuda", dtype=torch.float64) * s + (s - 1) / 2
    y, x = torch.meshgrid(ys, xs, indexing="ij")
    f = torch.stack([torch.stack(flow(x, y)) for flow in flows])
    gen = torch.Generator(device="cuda").manual_seed(7 + seed)
    return f + err * torch.randn(f.shape, generator=gen, device="cuda", dtype=torch.float64)


def _predictor(c, flows, seed):
    """What a predictor hands to the correlation: the flow to whole pixels."""
    return _nodes(c, flows, seed, 0.25).round().float()


def _upstream(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(99 + seed)
    return 0.5 + torch.rand((c["n"], c["h"] // 8, c["w"] // 8), generator=gen, device="cuda")


def prepare(case, seed):
    c = case
    A, B, flows = _frames(c, seed)
    s = dict(kind=c["kind"], A=A, B=B)
    if c["kind"] == "ssd":
        s["plan"] = api.Plan(c["w"], c["h"], max_batch=c["n"], dtype="f32", levels=1)
        s["U"] = _nodes(c, flows, seed, 0.2).float().requires_grad_(True)
        s["g"] = _upstream(c, seed)
        return s
    if c["kind"] == "preprocess":
        p = s["plan"] = api.Plan(c["w"], c["h"], max_batch=c["n"], dtype=c["dtype"], workspace=False)
        s.update(case=c, hp=torch.empty_like(A), cl=torch.empty_like(A),
                 lut=torch.empty(p.clahe_lut_bytes(c["n"], c["tiles_x"], c["tiles_y"]), dtype=torch.uint8,
                                 device="cuda"))
        return s
    p = s["plan"] = api.Plan(c["w"], c["h"], max_batch=c["n"], dtype=c["dtype"], win=c["win"], step=_step(c),
                             radius=c["radius"], levels=c["levels"], radius_coarse=c["rc"], radius_fine=c["rf"],
                             warp=c["warp"], peak=c["peak"], sgm=c["sgm"])
    f = lambda *k, t=torch.float32: torch.empty((c["n"], *k, p.ny, p.nx), dtype=t, device="cuda")  # noqa: E731
    s["out"] = dict(pred=f(2), disp=f(2), peak=f(), flags=f(t=torch.uint8), omega=f())
    if c["kind"] == "correct":
        s["pred"] = _predictor(c, flows, seed)
    return s


def run(state):
    s, p = state, state["plan"]
    if s["kind"] == "run":
        return p.run(s["A"], s["B"], s["out"])
    if s["kind"] == "predict":
        return p.predict(s["A"], s["B"], s["out"]["pred"])
    if s["kind"] == "correct":
        o = s["out"]
        return p.correct(s["A"], s["B"], s["pred"], o["disp"], o["peak"], o["flags"])
    if s["kind"] == "ssd":
        loss = autograd.warp_ssd(s["A"], s["B"], s["U"], p)
        return loss, torch.autograd.grad(loss, s["U"], s["g"])[0]
    c = s["case"]
    p.highpass(s["A"], s["hp"], radius=c["hp_radius"])
    p.clahe(s["hp"], s["cl"], tiles=(c["tiles_x"], c["tiles_y"]), clip_factor=c["clip"], lut=s["lut"])
    if c["dtype"] == "u16":   # (the same bytes: few torch operations take uint16)
        return s["hp"].view(torch.int16), s["cl"].view(torch.int16)
    return s["hp"], s["cl"]


def work(case):
    c = case
    es, n, px = {"u8": 1, "u16": 2, "f32": 4}[c["dtype"]], c["n"], c["n"] * c["w"] * c["h"]
    if c["kind"] == "preprocess":   # read, high-passed and equalised frame; per pixel a box mean, a count, a blend
        return dict(bytes=3.0 * px * es, flops=24.0 * px)
    vec = px / _step(c) ** 2
    if c["kind"] == "ssd":   # A, B, U, g in; loss, gradient out; per pixel two samples and the gradient's terms
        return dict(bytes=8.0 * px + vec * 4 * (2 + 1 + 1 + 2), flops=75.0 * px)
    # absolute differences of the block search, each pixel difference taken once for all blocks that share it
    sad = sum(2.0 * (px / 4 ** k) * (2 * (c["rc"] if k == c["levels"] - 1 else c["rf"]) + 1) ** 2 for k in range(c["levels"]))
    shifts = 5 if c["peak"] == "fixed" else (2 * c["radius"] + 1) ** 2
    warp = 40.0 if c["warp"] == "central" else 20.0
    corr = (2.0 * shifts + warp) * px + 25.0 * shifts * vec
    if c["kind"] == "predict":
        return dict(bytes=2.0 * px * es + 8 * vec, flops=sad)
    if c["kind"] == "correct":
        return dict(bytes=2.0 * px * es + (8 + 8 + 4 + 1) * vec, flops=corr)
    return dict(bytes=2.0 * px * es + (8 + 8 + 4 + 1 + 4) * vec, flops=sad + corr + 200.0 * vec)


# ---------------------------------------------------------------------------
# the same in 64 bits, plainly
# ---------------------------------------------------------------------------

def _interp(f, n, lo, hi, step, axis):
    """Node values along `axis` (n nodes at b step + (step-1)/2), linear, held
    outside, at the pixels lo..hi-1."""
    t = ((torch.arange(lo, hi, device=f.device, dtype=torch.float64) - (step - 1) / 2) / step).clamp(0, n - 1)
    b = t.floor().long().clamp(max=max(n - 2, 0))
    w = t - b
    w = w.reshape([-1] + [1] * (f.dim() - 1 - axis)) if axis < f.dim() - 1 else w
    return f.index_select(axis, b) * (1 - w) + f.index_select(axis, (b + 1).clamp(max=n - 1)) * w


def _dense(field, y0, y1, x0, x1, step):
    """[2][ny][nx] node field at the pixels of rows y0..y1-1, columns x0..x1-1."""
    return _interp(_interp(field.double(), field.shape[1], y0, y1, step, 1), field.shape[2], x0, x1, step, 2)


def _at(img, iy, ix):
    h, w = img.shape
    ok = (iy >= 0) & (iy < h) & (ix >= 0) & (ix < w)
    return torch.where(ok, img[iy.clamp(0, h - 1), ix.clamp(0, w - 1)], 0.0)


def _sample(img, y, x):
    """Bilinear, zero outside the image."""
    fy, fx = y.detach().floor(), x.detach().floor()
    iy, ix, ey, ex = fy.long(), fx.long(), y - fy, x - fx
    top = (1 - ex) * _at(img, iy, ix) + ex * _at(img, iy, ix + 1)
    bot = (1 - ex) * _at(img, iy + 1, ix) + ex * _at(img, iy + 1, ix + 1)
    return (1 - ey) * top + ey * bot


def _deformed(img, field, s, y0, y1, x0, x1, step):
    y = torch.arange(y0, y1, device="cuda", dtype=torch.float64)[:, None]
    x = torch.arange(x0, x1, device="cuda", dtype=torch.float64)[None, :]
    if field is None or s == 0.0:
        return _sample(img, y.expand(-1, x1 - x0), x.expand(y1 - y0, -1))
    u = s * _dense(field, y0, y1, x0, x1, step)
    return _sample(img, y + u[1], x + u[0])


def _cells(z, step):
    """Sums of the windows (2 step)^2 at spacing step of an image that starts
    at the first window."""
    h, w = z.shape
    s = z.reshape(h // step, step, w // step, step).sum((1, 3))
    s = s[:-1] + s[1:]
    return s[:, :-1] + s[:, 1:]


def _exact_correct(c, A, B, pred):
    """disp [2][ny][nx], peak of one pair."""
    st, R = _step(c), 1 if c["peak"] == "fixed" else c["radius"]
    h, H, W, n = st // 2, c["h"], c["w"], float(c["win"] ** 2)
    sa, sb = (-0.5, 0.5) if c["warp"] == "central" else (0.0, 1.0)
    K = float(A.double().mean().round())
    a = _deformed(A.double(), pred, sa, -h, H + h, -h, W + h, st) - K
    b = _deformed(B.double(), pred, sb, -h - R, H + h + R, -h - R, W + h + R, st) - K
    SA, VA = _cells(a, st), _cells(a * a, st)
    VA = VA - SA * SA / n
    G, rho = 2 * R + 1, {}
    hh, ww = a.shape
    for sy in range(-R, R + 1):
        for sx in range(-R, R + 1):
            if c["peak"] == "fixed" and sx and sy:
                continue
            z = b[R + sy:R + sy + hh, R + sx:R + sx + ww]
            SB, QB = _cells(z, st), _cells(z * z, st)
            VB = QB - SB * SB / n
            r = (_cells(a * z, st) - SA * SB / n) / torch.sqrt((VA * VB).clamp_min(1e-300))
            rho[sy, sx] = torch.where((VA > 1e-9) & (VB > 1e-6 * QB), r, 0.0)
    zero = torch.zeros_like(rho[0, 0])
    plane = torch.stack([rho.get((k // G - R, k % G - R), zero) for k in range(G * G)])
    by, bx = torch.zeros_like(zero, dtype=torch.long), torch.zeros_like(zero, dtype=torch.long)
    if c["peak"] != "fixed":
        best = torch.full_like(zero, -2.0)
        for sy, sx in sorted(rho, key=lambda k: (abs(k[0]) + abs(k[1]), k[0], k[1])):
            m = rho[sy, sx] > best
            best = torch.where(m, rho[sy, sx], best)
            by, bx = torch.where(m, sy, by), torch.where(m, sx, bx)

    def at(y, x):
        return plane.gather(0, ((y + R).clamp(0, G - 1) * G + (x + R).clamp(0, G - 1))[None])[0]

    def fit(m, o, p, edge):
        lm, l0, lp = (v.clamp_min(1e-3).log() for v in (m, o, p))
        den = 2 * (lm - 2 * l0 + lp)
        e = torch.where(den < 0, (lm - lp) / torch.where(den < 0, den, -1.0), 0.0)
        return e.clamp(-1, 1) if c["peak"] == "fixed" else torch.where(edge, 0.0, e)
    c0 = at(by, bx)
    ex = fit(at(by, bx - 1), c0, at(by, bx + 1), bx.abs() == R)
    ey = fit(at(by - 1, bx), c0, at(by + 1, bx), by.abs() == R)
    base = torch.zeros((2,) + zero.shape, dtype=torch.float64, device="cuda")
    if pred is not None:
        d = _dense(pred, -h, H + h, -h, W + h, st)
        base = torch.stack([_cells(d[0], st), _cells(d[1], st)]) / n
    return torch.stack([base[0] + bx + ex, base[1] + by + ey]), c0


def _neighbours(f, fill, centre=False):
    """The 3x3 neighbours [k][...] of the last two axes, `fill` outside."""
    p = torch.nn.functional.pad(f, (1, 1, 1, 1), value=fill)
    h, w = f.shape[-2:]
    return torch.stack([p[..., i:i + h, j:j + w] for i in range(3) for j in range(3) if centre or (i, j) != (1, 1)])


def _median(v, ok):
    """Median over axis 0 of the usable values, mean of the middle two."""
    k = ok.sum(0)
    s = torch.where(ok, v, math.inf).sort(0).values
    lo = s.gather(0, ((k - 1) // 2).clamp_min(0)[None])[0]
    hi = s.gather(0, (k // 2).clamp(max=v.shape[0] - 1)[None])[0]
    return torch.where(k > 0, 0.5 * (lo + hi), 0.0)


def _exact_validate(f, bad):
    """Normalised-median validation (threshold 2, 0.1 px) of f [2][ny][nx]."""
    ok = _neighbours((~bad).double(), 0.0) > 0
    out = bad.clone()
    for k in range(2):
        v = _neighbours(f[k], 0.0)
        med = _median(v, ok)
        out |= ((f[k] - med).abs() > 2.0 * (_median((v - med).abs(), ok) + 0.1)) & ok.any(0)
    good = _neighbours((~out).double(), 0.0) > 0
    return torch.stack([torch.where(out & good.any(0), _median(_neighbours(f[k], 0.0), good), f[k]) for k in range(2)])


def _exact_vorticity(f, h):
    return torch.gradient(f[1], spacing=float(h), dim=1, edge_order=2)[0] - \
        torch.gradient(f[0], spacing=float(h), dim=0, edge_order=2)[0]


def _low_median(f):
    """3x3 median inside the grid, the lower middle of an even count (integers)."""
    big = 1 << 20
    v = _neighbours(f, big, centre=True).sort(0).values
    return v.gather(0, ((v < big).sum(0) - 1).div(2, rounding_mode="floor")[None])[0]


def _block_sads(c, a, b, cx, cy, ny, nx, ds):
    """SAD of every node's block of a against b moved by centre + d for each d
    of ds: [len(ds)][ny][nx]."""
    st, w = _step(c), c["win"]
    lo, m = -(st // 2), 160
    pad = lambda z: torch.nn.functional.pad(z, (m, m + st, m, m + st))  # noqa: E731
    ap, bp = pad(a), pad(b)
    r = torch.arange(w, device="cuda")
    y = (torch.arange(ny, device="cuda") * st + lo + m)[:, None, None, None] + r[None, None, :, None]
    x = (torch.arange(nx, device="cuda") * st + lo + m)[None, :, None, None] + r[None, None, None, :]
    at = ap[y, x]
    yy, xx = y + cy[:, :, None, None], x + cx[:, :, None, None]
    return torch.stack([(at - bp[yy + dy, xx + dx]).abs().sum((2, 3)) for dy, dx in ds])


def _paths(cost, p1, p2):
    """Semi-global aggregation of cost [G][G][ny][nx] along the four paths."""
    total = torch.zeros_like(cost)
    for axis, back in ((3, False), (3, True), (2, False), (2, True)):
        z = cost.flip(axis) if back else cost
        out, prev = [], None
        for line in z.unbind(axis):
            if prev is None:
                cur = line
            else:
                q = torch.nn.functional.pad(prev.permute(2, 0, 1), (1, 1, 1, 1), value=1 << 40).permute(1, 2, 0)
                g = prev.shape[0]
                near = torch.stack([q[i:i + g, j:j + g] for i in range(3) for j in range(3) if (i, j) != (1, 1)]).amin(0)
                least = prev.amin((0, 1))
                cur = line + torch.minimum(torch.minimum(prev, near + p1), least + p2) - least
            out.append(cur)
            prev = cur
        z = torch.stack(out, axis)
        total += z.flip(axis) if back else z
    return total


def _exact_predict(c, A, B):
    """The integer predictor of one pair, [2][ny][nx] float64."""
    st, lv = _step(c), [(A.int(), B.int())]
    for _ in range(1, c["levels"]):
        def down(z):
            z = torch.nn.functional.pad(z, (0, z.shape[1] % 2, 0, z.shape[0] % 2))
            return (z[::2, ::2] + z[::2, 1::2] + z[1::2, ::2] + z[1::2, 1::2] + 2).div(4, rounding_mode="floor")
        lv.append(tuple(down(z) for z in lv[-1]))
    grids = [(c["h"] // st, c["w"] // st)]
    for _ in range(1, c["levels"]):
        grids.append(tuple((g + 1) // 2 for g in grids[-1]))
    f = None
    for k in range(c["levels"] - 1, -1, -1):
        (ny, nx), coarse = grids[k], k == c["levels"] - 1
        R = c["rc"] if coarse else c["rf"]
        if coarse:
            cx = cy = torch.zeros((ny, nx), dtype=torch.long, device="cuda")
        else:
            ya, xa = (torch.arange(ny, device="cuda") // 2)[:, None], (torch.arange(nx, device="cuda") // 2)[None, :]
            cx, cy = 2 * f[0][ya, xa], 2 * f[1][ya, xa]
        ds = [(dy, dx) for dy in range(-R, R + 1) for dx in range(-R, R + 1)]
        sad = _block_sads(c, *lv[k], cx, cy, ny, nx, ds).long()
        if coarse and c["sgm"]:
            G, bb = 2 * R + 1, c["win"] ** 2
            sad = _paths(sad.reshape(G, G, ny, nx), 2 * bb, 16 * bb).reshape(G * G, ny, nx)
        d = torch.tensor(ds, device="cuda")
        dy, dx = d[:, 0][:, None, None] + cy, d[:, 1][:, None, None] + cx
        key = (((sad << 8) + dx.abs() + dy.abs()) << 16) + ((dy + 128) << 8) + dx + 128
        best = key.amin(0)
        f = torch.stack([(best & 255) - 128, ((best >> 8) & 255) - 128])
        f = torch.stack([_low_median(f[0]), _low_median(f[1])])
    return f.double()


def _exact_ssd(c, A, B, U, g):
    """(loss, gradient) of one pair."""
    h, H, W = 4, c["h"], c["w"]
    U = U.detach().double().requires_grad_(True)
    with torch.enable_grad():
        r = _deformed(B.double(), U, 1.0, -h, H + h, -h, W + h, 8) - _deformed(A.double(), None, 0.0, -h, H + h, -h, W + h, 8)
        loss = _cells(r * r, 8)
        grad = torch.autograd.grad(loss, U, g.double())[0]
    return loss.detach(), grad


def exact(case, seed):
    c = case
    if c["kind"] == "preprocess":   # whole numbers
        return None
    A, B, flows = _frames(c, seed)
    n = c["n"]
    with torch.no_grad():
        if c["kind"] == "ssd":
            U, g = _nodes(c, flows, seed, 0.2).float(), _upstream(c, seed)
            got = [_exact_ssd(c, A[i], B[i], U[i], g[i]) for i in range(n)]
            return torch.stack([x[0] for x in got]), torch.stack([x[1] for x in got])
        if c["kind"] == "correct":
            pred = _predictor(c, flows, seed)
            got = [_exact_correct(c, A[i], B[i], pred[i]) for i in range(n)]
            return torch.stack([x[0] for x in got]), torch.stack([x[1] for x in got]), None
        pred = [_exact_predict(c, A[i], B[i]) for i in range(n)]
        if c["kind"] == "predict":
            return torch.stack(pred)
        res = dict(pred=[], disp=[], peak=[], omega=[])
        none = torch.zeros(pred[0].shape[1:], dtype=torch.bool, device="cuda")
        R = 1 if c["peak"] == "fixed" else c["radius"]
        for i in range(n):
            p = _exact_validate(pred[i], none)
            d, peak = _exact_correct(c, A[i], B[i], p)
            edge = none
            if c["peak"] != "fixed":   # best shift on the edge of the search: not a measurement
                h = _step(c) // 2
                m = _dense(p, -h, c["h"] + h, -h, c["w"] + h, _step(c))
                s = torch.stack([d[k] - _cells(m[k], _step(c)) / c["win"] ** 2 for k in range(2)])
                edge = (s.abs() >= R - 1e-9).any(0)
            d = _exact_validate(d, edge)
            for k, v in (("pred", p), ("disp", d), ("peak", peak), ("omega", _exact_vorticity(d, _step(c)))):
                res[k].append(v)
        out = {k: torch.stack(v) for k, v in res.items()}
        out["flags"] = None
        return out
