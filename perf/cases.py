"""The work that users of this library have it do, as cases that can be timed.

listed() names them, draw() gives more of the same ranges, prepare() makes what
a program holds before the call (inputs on the GPU, the context it keeps),
run() is one pass through the public calls, work() what such a pass cannot do
without, and exact() the same result from plain torch and numpy in 64 bits.

Kinds of case:
  project  full Dykstra on one image (Context.project), the library's main call
  batch    full Dykstra on images of different sizes (Context.project_batch)
  icd      the paper's incomplete Dykstra on an image or on a movie's frames
  nested   incomplete Dykstra over a divisor chain of square sides
  admm     the ADMM deblurring loop around either projection
  mc       the Monte-Carlo statistic that balances the window bounds
"""
import math
import random

import numpy as np
import torch

import paper_1503_03492_amd as smre

PIXELS_PER_EMITTER = 1300.0   # density of the batch and serving images
PSF = 1.5                     # width of an emitter, pixels


def listed():
    return [
        # the smallest solve a user runs: a 64 x 64 image in FP64, three sides;
        # launches and latency are all it costs
        dict(name="project_64_f64", kind="project", H=64, W=64, smin=1, smax=4, step=0,
             dtype="f64", inc="same", scene="noise", tol=1e-10, sweeps=200),
        # an image of odd size with plain noise in it
        dict(name="project_203x317_f32", kind="project", H=203, W=317, smin=1, smax=8, step=1,
             dtype="f32", inc="same", scene="noise", tol=1e-6, sweeps=100),
        # a fluorescence frame at the size and sides of the 512 x 512 benchmark
        dict(name="project_512_f32", kind="project", H=512, W=512, smin=1, smax=8, step=1,
             dtype="f32", inc="same", scene="emitters", tol=1e-5, sweeps=120),
        # the benchmark image: 1024 x 1024, sides 1..16, the first sweeps of a solve
        dict(name="project_1024_f32", kind="project", H=1024, W=1024, smin=1, smax=16, step=1,
             dtype="f32", inc="same", scene="emitters", tol=1e-5, sweeps=100),
        # the same image with increments kept in BF16
        dict(name="project_1024_bf16", kind="project", H=1024, W=1024, smin=1, smax=16, step=1,
             dtype="f32", inc="bf16", scene="emitters", tol=1e-5, sweeps=60),
        # a batch of uneven frames in one call
        dict(name="batch_16_uneven_f32", kind="batch", n=16, lo=128, hi=768, pick=1, smax=8,
             dtype="f32", tol=1e-5, sweeps=60),
        # the paper's incomplete Dykstra on one large frame, its stopping rule
        dict(name="icd_1024_f32", kind="icd", H=1024, W=1024, frames=1, K=4, dtype="f32",
             mode="mean", tol=1e-3),
        # the frames of a blinking movie, all in one call (the largest input)
        dict(name="icd_movie_512_f32", kind="icd", H=512, W=512, frames=1000, K=4, dtype="f32",
             mode="mean", tol=1e-3),
        # hierarchies that are not powers of two
        dict(name="nested_48_1024_f32", kind="nested", H=1024, W=1024, chain="1,3,6,12,24,48",
             dtype="f32", mode="mean", tol=1e-3),
        # deblurring a photograph-like scene, incomplete projection in the loop
        dict(name="admm_512_icd_f32", kind="admm", H=512, W=512, method="icd", K=4, sigma=4.0,
             iters=20, dtype="f32", smax=16, sweeps=1),
        # the same loop with the exact projection, its increments kept between
        # iterations: grey levels far outside the bounds, many windows active
        dict(name="admm_256_full_f32", kind="admm", H=256, W=256, method="full", K=4, sigma=2.0,
             iters=3, dtype="f32", smax=8, sweeps=40),
        # the bounds' quantile statistic from drawn fields
        dict(name="mc_1024_sides16", kind="mc", H=1024, W=1024, smax=16, fields=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["project"] * 4 + ["batch", "icd", "icd", "nested", "admm", "mc"])
    if kind == "project":
        H, W = _log(rng, 48, 1024), _log(rng, 48, 1024)
        smax = rng.randint(3, 16)
        dtype = rng.choice(["f32", "f32", "f64"])
        inc = "bf16" if dtype == "f32" and rng.random() < 0.25 else "same"
        return dict(kind=kind, H=H, W=W, smin=rng.choice([1, 1, 2]), smax=smax,
                    step=rng.choice([0, 1, 1]), dtype=dtype, inc=inc,
                    scene=rng.choice(["noise", "emitters", "emitters"]), tol=1e-6,
                    sweeps=_log(rng, 10, 50))
    if kind == "batch":
        return dict(kind=kind, n=rng.randint(2, 12), lo=rng.randint(64, 160),
                    hi=rng.randint(256, 640), pick=rng.randint(2, 10 ** 6), smax=rng.randint(4, 12),
                    dtype=rng.choice(["f32", "f32", "f64"]), tol=1e-5, sweeps=_log(rng, 8, 30))
    if kind == "icd":
        frames = rng.choice([1, 1, _log(rng, 2, 200)])
        side = 2048 if frames == 1 else 512
        return dict(kind=kind, H=_log(rng, 64, side), W=_log(rng, 64, side), frames=frames,
                    K=rng.randint(2, 5), dtype=rng.choice(["f32", "f32", "f64"]),
                    mode=rng.choice(["mean", "mean", "max"]), tol=1e-3)
    if kind == "nested":
        return dict(kind=kind, H=_log(rng, 96, 1024), W=_log(rng, 96, 1024),
                    chain=rng.choice(["1,3,6", "1,3,6,12,24,48", "1,2,4,8,16,32,64", "2,6,12",
                                      "1,2,6,24"]),
                    dtype=rng.choice(["f32", "f64"]), mode=rng.choice(["mean", "max"]), tol=1e-3)
    if kind == "admm":
        method = rng.choice(["icd", "icd", "full"])
        top = 640 if method == "icd" else 256
        return dict(kind=kind, H=_log(rng, 96, top), W=_log(rng, 96, top), method=method,
                    K=rng.randint(2, 4), sigma=round(rng.uniform(1.0, 5.0), 2),
                    iters=rng.randint(4, 20) if method == "icd" else 2,
                    dtype=rng.choice(["f32", "f32", "f64"]), smax=rng.randint(4, 8),
                    sweeps=rng.randint(10, 30))
    return dict(kind="mc", H=_log(rng, 64, 1024), W=_log(rng, 64, 1024), smax=rng.randint(4, 24),
                fields=_log(rng, 8, 128))


# ---------------------------------------------------------------- what a case means
def _sides(case):
    """Window sides of a full projection: every side, or powers of two (step 0)."""
    if case.get("step", 1) == 0:
        top = [s for s in (1, 2, 4, 8, 16) if case["smin"] <= s <= case["smax"]]
    else:
        top = list(range(case["smin"], case["smax"] + 1))
    return [s for s in top if s <= min(case.get("H", 64), case.get("W", 64))]


def _chain(case):
    if case["kind"] == "nested":
        return [int(s) for s in case["chain"].split(",")]
    return [1 << k for k in range(case["K"] + 1)]


def _phases(chain):
    """The paper's pattern: phase i shifts both axes by side[i] (modulo the
    block) and projects the levels from i up."""
    return [(s % chain[-1], s % chain[-1], i) for i, s in enumerate(chain)]


def _batch_sizes(case):
    pick = random.Random(case["pick"])
    sizes = (128, 256, 384, 512, 768)
    fixed = [s for s in sizes if case["lo"] <= s <= case["hi"]]
    if case["lo"] == 128 and case["hi"] == 768:
        return [(s, s) for s in (pick.choice(fixed) for _ in range(case["n"]))]
    return [(_log(pick, case["lo"], case["hi"]), _log(pick, case["lo"], case["hi"]))
            for _ in range(case["n"])]


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


# ---------------------------------------------------------------- inputs
def _blur(x, sigma, radius=None):
    """Gaussian blur of the last two axes, zero outside, taps cut at radius."""
    r = int(4.0 * sigma + 0.5) if radius is None else radius
    if sigma == 0:
        return x
    w = torch.exp(-0.5 * (torch.arange(-r, r + 1, dtype=torch.float64) / sigma) ** 2)
    w = (w / w.sum()).tolist()
    for axis in (-1, -2):
        n = x.shape[axis]
        pad = [r, r] if axis == -1 else [0, 0, r, r]
        p = torch.nn.functional.pad(x, pad)
        out = torch.zeros_like(x)
        for k, wk in enumerate(w):
            out += wk * p.narrow(axis, k, n)
        x = out
    return x


def _emitters(gen, H, W, n_e=None):
    """Residual of a fluorescence frame: point emitters with Poisson counts,
    blurred, minus the blurred mean, in units of its standard deviation."""
    n_e = max(1, int(round(H * W / (PIXELS_PER_EMITTER if n_e is None else n_e))))
    at = torch.randint(0, H * W, (n_e,), generator=gen)
    counts = torch.poisson(torch.full((n_e,), 50.0, dtype=torch.float64), generator=gen)
    E = torch.zeros(H * W, dtype=torch.float64).index_add_(0, at, counts - 50.0)
    R = _blur(E.view(H, W).cuda(), PSF)
    sd = float(R.std(correction=0))
    return R / sd if sd > 0 else R


def _noise(gen, H, W):
    """Unit noise with one bright spot in the middle."""
    x = torch.randn(H, W, generator=gen, dtype=torch.float64)
    r = torch.arange(H, dtype=torch.float64)[:, None] - (H - 1) / 2.0
    c = torch.arange(W, dtype=torch.float64)[None, :] - (W - 1) / 2.0
    return (x + 4.0 * torch.exp(-(r * r + c * c) / 18.0)).cuda()


def _scene(gen, H, W, sigma):
    """A grey-level scene of smooth shading, ellipses and boxes, blurred, plus
    unit noise: the data of a deblurring problem."""
    yy = (torch.arange(H, dtype=torch.float64) / max(H - 1, 1))[:, None].expand(H, W)
    xx = (torch.arange(W, dtype=torch.float64) / max(W - 1, 1))[None, :].expand(H, W)
    img = 60.0 + 60.0 * yy + 40.0 * xx
    for _ in range(40):
        cy, cx, ry, rx, level, box = torch.rand(6, generator=gen, dtype=torch.float64).tolist()
        ry, rx = 0.03 + 0.22 * ry, 0.03 + 0.22 * rx
        if box < 0.5:
            mask = ((yy - cy) / ry) ** 2 + ((xx - cx) / rx) ** 2 <= 1.0
        else:
            mask = ((yy - cy).abs() <= ry) & ((xx - cx).abs() <= rx)
        img = torch.where(mask, 255.0 * level, img)
    img = _blur(img.clamp(0.0, 255.0).cuda(), sigma)
    return img + torch.randn(H, W, generator=gen, dtype=torch.float64).cuda()


def _movie(gen, frames, H, W, dtype):
    """Fluctuations of blinking emitters about their mean counts: on and off
    times from a power law, Poisson counts while on."""
    n_e = max(1, int(round(H * W / PIXELS_PER_EMITTER)))
    at = torch.randint(0, H * W, (n_e,), generator=gen)
    tau = torch.ceil(torch.rand(n_e, frames, generator=gen, dtype=torch.float64).clamp_min(1e-9)
                     ** -2.0)
    flips = torch.cumsum(tau, 1)
    t = torch.arange(frames, dtype=torch.float64).expand(n_e, frames).contiguous()
    on = (torch.searchsorted(flips, t, right=True)
          + torch.randint(0, 2, (n_e, 1), generator=gen)) % 2
    counts = torch.poisson(torch.full((n_e, frames), 50.0), generator=gen) * on
    fluct = (counts - counts.mean(1, keepdim=True)).cuda().to(dtype)
    at = at.cuda()
    out = torch.empty(frames, H, W, dtype=dtype, device="cuda")
    for f in range(0, frames, 200):
        m = min(200, frames - f)
        E = torch.zeros(H * W, m, dtype=dtype, device="cuda")
        E.index_add_(0, at, fluct[:, f:f + m])
        out[f:f + m] = _blur(E.t().contiguous().view(m, H, W), PSF)
    return out / out.std().clamp_min(1e-12)


def _input(case, seed):
    gen = torch.Generator().manual_seed(int(seed))
    dt = _dtype(case) if "dtype" in case else torch.float64
    if case["kind"] == "project":
        if case["scene"] == "noise":
            return _noise(gen, case["H"], case["W"]).to(dt)
        # the benchmark frames: 2000 emitters on 1024 x 1024, 200 on 512 x 512
        return _emitters(gen, case["H"], case["W"],
                         524.3 if case["smax"] > 8 else 1310.7).to(dt)
    if case["kind"] == "batch":
        return [_emitters(gen, h, w).to(dt) for h, w in _batch_sizes(case)]
    if case["kind"] == "icd" and case["frames"] > 1:
        return _movie(gen, case["frames"], case["H"], case["W"], dt)
    if case["kind"] in ("icd", "nested"):
        return _emitters(gen, case["H"], case["W"], 524.3).to(dt)
    return _scene(gen, case["H"], case["W"], case["sigma"]).to(dt)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, ctx=smre.Context(0))
    if kind == "mc":
        st["sides"] = _sides(dict(case, smin=1))
        st["seed"] = int(seed)
        return st
    st["x0"] = _input(case, seed)
    if kind == "project":
        st["sides"] = _sides(case)
    elif kind == "batch":
        st["sides"] = list(range(1, case["smax"] + 1))
    elif kind == "admm":
        st["sides"] = list(range(1, case["smax"] + 1))
        st["r2_icd"] = smre.chi2_bounds([1 << k for k in range(case["K"] + 1)])
    else:
        st["sides"] = _chain(case)
    st["r2"] = smre.chi2_bounds(st["sides"])
    if kind == "batch":
        st["x"] = [torch.empty_like(x) for x in st["x0"]]
    elif kind != "admm":
        st["x"] = torch.empty_like(st["x0"])
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "project":
        x = st["x"].copy_(st["x0"])     # the projection works in place
        inc = smre.INC_BF16 if case["inc"] == "bf16" else smre.INC_SAME
        _, rep = ctx.project(x, st["sides"], st["r2"], tol=case["tol"],
                             max_sweeps=case["sweeps"], inc=inc)
        return {"x": x, "max_violation": rep["max_violation"], "sweeps": rep["sweeps"]}
    if kind == "batch":
        for x, x0 in zip(st["x"], st["x0"]):
            x.copy_(x0)
        _, reps = ctx.project_batch(st["x"], st["sides"], st["r2"], tol=case["tol"],
                                    max_sweeps=case["sweeps"], region=16)
        return {"x": st["x"], "max_violation": [r["max_violation"] for r in reps]}
    if kind == "admm":
        if case["method"] == "icd":
            x, eps, rep = ctx.admm(st["x0"], case["sigma"], K=case["K"],
                                   radius2_icd=st["r2_icd"], delta=-1.0, max_iter=case["iters"],
                                   want_eps=True)
        else:
            x, eps, rep = ctx.admm(st["x0"], case["sigma"], method=smre.ADMM_FULL,
                                   sides=st["sides"], radius2=st["r2"], full_tol=1e-6,
                                   full_max_sweeps=case["sweeps"], full_warm=True, delta=-1.0,
                                   max_iter=case["iters"], want_eps=True)
        return {"x": x, "eps": eps, "residual": rep["last_residual"],
                "iterations": rep["iterations"]}
    if kind == "mc":
        q, tmax, _ = ctx.mc_statistic(case["H"], case["W"], st["sides"], st["seed"],
                                      case["fields"], want_tmax=True)
        return {"q": q, "tmax": tmax}
    x = st["x"].copy_(st["x0"])
    mode = smre.TOL_MEANABS if case["mode"] == "mean" else smre.TOL_MAXABS
    if kind == "nested":
        rep = ctx.incomplete_nested(x, st["sides"], st["r2"], _phases(st["sides"]),
                                    tol=case["tol"], mode=mode)
    elif case["frames"] > 1:
        rep = ctx.incomplete_frames(x, case["K"], st["r2"], tol=case["tol"], mode=mode)
    else:
        rep = ctx.incomplete(x, case["K"], st["r2"], tol=case["tol"], mode=mode)
    return {"x": x, "max_violation": rep["max_violation"]}


# ---------------------------------------------------------------- what a pass cannot do without
def _windows(H, W, sides):
    return sum((H - s + 1) * (W - s + 1) for s in sides if s <= min(H, W))


def work(case):
    """Inputs read once and results written once; the operations: a full
    projection has to test every window once per sweep (four operations with
    running sums), an incomplete one its squares at least once per phase (two
    per pixel and level), the statistic has a square per pixel and four per
    window, a blur pass 2 (2 R + 1) per pixel."""
    b = 8 if case.get("dtype") == "f64" else 4
    kind = case["kind"]
    if kind == "project":
        HW = case["H"] * case["W"]
        return {"bytes": 2 * b * HW,
                "flops": 4 * case["sweeps"] * _windows(case["H"], case["W"], _sides(case))}
    if kind == "batch":
        sizes, sides = _batch_sizes(case), range(1, case["smax"] + 1)
        return {"bytes": 2 * b * sum(h * w for h, w in sizes),
                "flops": 4 * case["sweeps"] * sum(_windows(h, w, sides) for h, w in sizes)}
    if kind in ("icd", "nested"):
        n = case["H"] * case["W"] * case.get("frames", 1)
        lv = len(_chain(case))
        return {"bytes": 2 * b * n, "flops": 2 * n * lv * (lv + 1) // 2}
    if kind == "admm":
        HW = case["H"] * case["W"]
        taps = 2 * int(4.0 * case["sigma"] + 0.5) + 1
        per = 8 * taps + 20
        if case["method"] == "icd":
            per += (case["K"] + 1) * (case["K"] + 2)
            proj = 0
        else:
            proj = 4 * case["sweeps"] * _windows(case["H"], case["W"],
                                                 range(1, case["smax"] + 1))
        return {"bytes": 3 * b * HW, "flops": case["iters"] * (per * HW + proj)}
    HW = case["H"] * case["W"]
    return {"bytes": 8 * case["fields"] * (1 + case["smax"]),
            "flops": case["fields"] * (HW + 4 * _windows(case["H"], case["W"],
                                                         range(1, case["smax"] + 1)))}


# ---------------------------------------------------------------- the same in 64 bits
def _box(x, s):
    c = torch.nn.functional.pad(x.cumsum(-1).cumsum(-2), (1, 0, 1, 0))
    return c[..., s:, s:] - c[..., :-s, s:] - c[..., s:, :-s] + c[..., :-s, :-s]


def _violation(x, sides, r2):
    x2 = x * x
    H, W = x.shape[-2:]
    return max([float(_box(x2, s).max()) / float(r) - 1.0
                for s, r in zip(sides, r2) if s <= min(H, W)])


class _Full64:
    """Dykstra over every window in the library's default visiting order:
    anchor regions of 16 x 16 in four colours, sides descending, offsets in
    raster order."""

    def __init__(self, H, W, sides, r2):
        self.steps, R = [], 16
        order = sorted(zip(sides, r2), reverse=True)

        def anchors(n, s, par, off):
            at = [a for p in range(par, (n + R - 1) // R, 2)
                  for a in range(p * R + off, min(p * R + R, n - s + 1), s)]
            return torch.tensor(at, dtype=torch.long, device="cuda")

        for cy in (0, 1):
            for cx in (0, 1):
                for s, r in order:
                    win = torch.arange(s, device="cuda")
                    rows = [anchors(H, s, cy, a) for a in range(min(s, R))]
                    cols = [anchors(W, s, cx, b) for b in range(min(s, R))]
                    for ra in rows:
                        for cb in cols:
                            if len(ra) and len(cb):
                                i = (ra[:, None] + win)[:, None, :, None]
                                j = (cb[:, None] + win)[None, :, None, :]
                                self.steps.append((i * W + j, float(r)))
        self.q = None

    def solve(self, x, sweeps, warm=False):
        H, W = x.shape
        x0 = x.clone()
        if not warm:
            self.q = [torch.zeros(i.shape, dtype=torch.float64, device="cuda")
                      for i, _ in self.steps]
        else:
            x = x - self.total
        x = x.reshape(-1).clone()
        for _ in range(sweeps):
            for k, (at, r) in enumerate(self.steps):
                y = x[at] + self.q[k]
                n = (y * y).sum((2, 3), keepdim=True)
                z = y * (r / torch.clamp_min(n, r)).sqrt()
                x[at] = z
                self.q[k] = y - z
        x = x.view(H, W)
        self.total = x0 - x
        return x


def _icd64(x, chain, r2, phases, tol, mean, max_inner=10000):
    """Incomplete Dykstra of one image: blocks of the largest side, each until
    its own stopping rule holds."""
    H, W = x.shape
    B = chain[-1]
    for sy, sx, lo in phases:
        oy, ox = (sy - B if sy else 0), (sx - B if sx else 0)
        nby, nbx = -((oy - H) // B), -((ox - W) // B)
        pad = torch.zeros(nby * B, nbx * B, dtype=torch.float64, device="cuda")
        inside = torch.zeros_like(pad)
        pad[-oy:H - oy, -ox:W - ox] = x
        inside[-oy:H - oy, -ox:W - ox] = 1.0

        def blocks(p):
            return p.view(nby, B, nbx, B).permute(0, 2, 1, 3).reshape(-1, B, B)

        xb, npix = blocks(pad).clone(), blocks(inside).sum((1, 2))
        levels = []
        for j in range(len(chain) - 1, lo - 1, -1):
            L = chain[j]
            full = blocks(inside).reshape(-1, B // L, L, B // L, L).sum((2, 4)) == L * L
            levels.append([L, float(r2[j]), full])
        live = torch.arange(xb.shape[0], device="cuda")
        v, q = xb, [torch.zeros_like(xb) for _ in levels]
        full = [f for _, _, f in levels]
        for _ in range(max_inner):
            moved = torch.zeros(v.shape[0], dtype=torch.float64, device="cuda")
            for k, (L, r, _) in enumerate(levels):
                y = v + q[k]
                n = (y * y).view(-1, B // L, L, B // L, L).sum((2, 4))
                t = torch.where(full[k] & (n > r), (r / torch.clamp_min(n, r)).sqrt(),
                                torch.ones_like(n))
                z = y * t.repeat_interleave(L, 1).repeat_interleave(L, 2)
                d = (v - z).abs()
                moved = moved + d.sum((1, 2)) if mean else torch.maximum(moved, d.amax((1, 2)))
                q[k], v = y - z, z
            stop = moved <= tol * npix[live] if mean else moved < tol
            if bool(stop.any()):
                xb[live[stop]] = v[stop]
                go = ~stop
                live, v = live[go], v[go]
                q, full = [a[go] for a in q], [f[go] for f in full]
            if not len(live):
                break
        xb[live] = v
        p = xb.view(nby, nbx, B, B).permute(0, 2, 1, 3).reshape(nby * B, nbx * B)
        x = p[-oy:H - oy, -ox:W - ox].clone()
    return x


def _admm64(case, I, r2_icd, sides, r2):
    lam, rho1, rho2, a1, a2 = 1.0, 6.192, 1.8, 1.2, 0.12
    gamma, sigma = 0.5 * (rho1 + rho2), case["sigma"]
    x, z, eps, Y1, Y2 = (torch.zeros_like(I) for _ in range(5))
    Ax = _blur(x, sigma)
    chain = _chain(dict(kind="icd", K=case["K"]))
    full = _Full64(*I.shape, sides, r2) if case["method"] == "full" else None
    for it in range(case["iters"]):
        t = rho1 * (I - Ax - eps) + Y1
        x = x - (-_blur(t, sigma) + rho2 * (x - z) + Y2) / (2.0 * gamma)
        Ax = _blur(x, sigma)
        e = I - Ax + Y1 / rho1
        if full is None:
            eps = _icd64(e, chain, r2_icd, _phases(chain), 1e-3, True)
        else:
            eps = full.solve(e, case["sweeps"], warm=it > 0)
        z = (rho2 * x + Y2) / (lam + rho2)
        res = I - Ax - eps
        Y1, Y2 = Y1 + a1 * res, Y2 + a2 * (x - z)
    return {"x": x, "eps": eps, "residual": float(res.norm()), "iterations": None}


def _mc64(case, sides, seed):
    H, W = case["H"], case["W"]
    npix = H * W
    ng = (npix + 3) // 4
    T = np.empty((case["fields"], len(sides)))
    for f in range(case["fields"]):
        # numpy advances the 256-bit counter before it generates a block
        c = (f << 64) - 1 if f else (1 << 256) - 1
        ctr = np.array([(c >> (64 * k)) & (2 ** 64 - 1) for k in range(4)], dtype=np.uint64)
        bits = np.random.Philox(key=np.array([seed, 0], dtype=np.uint64), counter=ctr)
        w = (bits.random_raw(4 * ng) >> np.uint64(11)).astype(np.int64)
        u = (torch.from_numpy(w).cuda().double() + 0.5) * 2.0 ** -53
        u = u.view(-1, 2)
        r, ang = (-2.0 * u[:, 0].log()).sqrt(), 2.0 * math.pi * u[:, 1]
        e = torch.stack([r * ang.cos(), r * ang.sin()], 1).reshape(-1)[:npix].view(H, W)
        e2 = e * e
        T[f] = torch.stack([_box(e2, s).max() for s in sides]).cpu().numpy()
    s = np.array(sides, dtype=np.float64)
    Q = ((T ** 0.25 - (s * s - 0.5) ** 0.25) * np.sqrt(8.0 * s)).max(1)
    return {"q": Q, "tmax": T}


def exact(case, seed):
    kind = case["kind"]
    if kind == "mc":
        if case["fields"] * case["H"] * case["W"] > 1.5e8:
            return None
        return _mc64(case, _sides(dict(case, smin=1)), int(seed))
    x0 = _input(case, seed)
    if kind in ("project", "batch"):
        sides = _sides(case) if kind == "project" else list(range(1, case["smax"] + 1))
        r2 = _chi2(sides)
        many = case["n"] if kind == "batch" else 1
        steps = 4 * sum(s * s for s in sides) * case["sweeps"] * many
        pixels = steps * 0.25 * (case["H"] * case["W"] if kind == "project" else 1e5)
        if case.get("inc") == "bf16" or steps * 1.1e-4 + pixels * 4e-10 > 15.0:
            return None
        xs = []
        for x in (x0 if kind == "batch" else [x0]):
            xs.append(_Full64(*x.shape, sides, r2).solve(x.double(), case["sweeps"]))
        if kind == "batch":
            return {"x": xs, "max_violation": [_violation(x, sides, r2) for x in xs]}
        return {"x": xs[0], "max_violation": _violation(xs[0], sides, r2), "sweeps": None}
    if kind == "admm":
        if case["method"] == "full":
            steps = 4 * sum(s * s for s in range(1, case["smax"] + 1)) * case["sweeps"]
            if steps * case["iters"] * 1.1e-4 > 15.0:
                return None
        sides = list(range(1, case["smax"] + 1))
        return _admm64(case, x0.double(), _chi2([1 << k for k in range(case["K"] + 1)]),
                       sides, _chi2(sides))
    chain = _chain(case)
    r2 = _chi2(chain)
    frames = case.get("frames", 1)
    if frames * case["H"] * case["W"] > 3e7 or frames > 60:
        return None
    xs = [_icd64(x.double(), chain, r2, _phases(chain), case["tol"], case["mode"] == "mean")
          for x in (x0 if frames > 1 else x0[None])]
    out = torch.stack(xs)
    return {"x": out if frames > 1 else out[0], "max_violation": _violation(out, chain, r2)}


def _chi2(sides, p=0.9):
    """Chi-square p-quantiles with s^2 degrees of freedom, by bisection on the
    regularised incomplete gamma function."""
    out = []
    for s in sides:
        a = torch.tensor(0.5 * s * s, dtype=torch.float64)
        lo, hi = 0.0, 4.0 * s * s + 100.0
        for _ in range(200):
            mid = 0.5 * (lo + hi)
            if float(torch.special.gammainc(a, torch.tensor(0.5 * mid, dtype=torch.float64))) < p:
                lo = mid
            else:
                hi = mid
        out.append(0.5 * (lo + hi))
    return out
