"""The work that users have this library do, as cases that can be timed.

Each case names one use of the public entry points in
`paper_1901_02492_amd.lib` with its sizes:

  step        images -> likelihood planes -> search -> ordered top-k of one
              stack (`run_search`), float32 or with 16-bit planes and the
              float32 re-score, with the bright-pixel mask before it where the
              workload has one
  serve       several stacks of uneven shape: planes of each, one batched
              search, ordered top-k of each
  threshold   planes, every trajectory above a level, their duplicates grouped
  cluster     the grouping alone, on a long hit list
  lightcurve  the light-curve outlier filter over every pixel's candidates
  stamps      coadded postage stamps and the moment filter
  planes      the likelihood planes alone, with their 16-bit copy or without

Inputs follow the paper's data as `paper_1901_02492_amd/synth.py` describes
it: sky noise with a smooth sigma of 0.8 to 1.2, variance sigma^2, 1% masked
pixels, moving sources, single-image flashes, visits 0.06 d apart on
consecutive nights, a Gaussian PSF.  They are drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

from paper_1901_02492_amd import lib

DEV = "cuda:0"
NU_MIN = 10.0                        # threshold mode's level
EPS = 4.0                            # clustering radius in pixels
SIGMA_CUT = 5.0                      # light-curve filter
STAMP_LIMITS = (0.5, 1.5, 0.5, 6.0)  # max_offset, max_m11, m2_min, m2_max
MAX_HITS = 1 << 20                   # hit list of the threshold mode
EXACT_TIE = 5e10                     # largest search whose scores exact() computes


# ---------------------------------------------------------------------------
# The cases.
# ---------------------------------------------------------------------------

def _step(name, n, h, w, speeds, angles, k, kc=None, lp="", grid="survey", psf=11):
    c = dict(kind="step", n=n, h=h, w=w, speeds=speeds, angles=angles, k=k, kc=kc or k, lp=lp,
             grid=grid, psf=psf)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest whole call: the 5 x 64^2 stack of the tests and the
        # smoke run, 121 velocities, 5 kept.  Launches and host work count.
        _step("step_small", 5, 64, 64, 11, 11, 5, grid="box", psf=7),
        # A cut-out searched around a known object: few tiles, a full-length
        # list, sizes that divide nothing.
        _step("step_cutout", 12, 251, 301, 20, 20, 50),
        # The flagship step: 15 x 4096^2, 600 velocities, 50 kept, float32.
        _step("step_survey", 15, 4096, 4096, 25, 24, 50),
        # The paper's dense velocity grid (250 speeds x 128 angles) with its
        # bright-pixel mask, on a quarter-width patch.
        _step("step_hits", 13, 1024, 1024, 250, 128, 50, grid="hits"),
        # The large-stack step in its 16-bit mode: 25 images, 4000 velocities.
        _step("step_large_f16", 25, 1024, 2048, 50, 80, 50, lp="f16"),
        # 16-bit mode in bfloat16 with its over-fetch of 2, one ragged frame
        # of few images.
        _step("step_ragged_bf16", 9, 613, 1187, 13, 20, 50, kc=52, lp="bf16"),
        # Serving: six small uneven stacks share one batched launch.
        dict(name="serve_small", kind="serve", jobs=6, shapes=1, k=50, lp=""),
        # Threshold mode (nu >= 10) on the survey recipe and its clustering.
        dict(name="threshold", kind="threshold", n=15, h=2048, w=2048, speeds=25, angles=24),
        # Clustering of a long hit list.
        dict(name="cluster", kind="cluster", hits=4_000_000),
        # The filter over the top 50 of every start pixel.
        dict(name="lightcurve", kind="lightcurve", n=15, h=1024, w=1024, k=50, q=1.0),
        # Stamps of 262144 candidates, radius 5.
        dict(name="stamps", kind="stamps", n=15, h=2048, w=2048, cands=262144, radius=5),
        # Planes with their half-precision copy.
        dict(name="planes_f16", kind="planes", n=20, h=2048, w=2048, psf=11, lp="f16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "serve", "threshold", "cluster", "lightcurve",
                       "stamps", "planes"])
    if kind == "step":
        grid = rng.choice(["survey", "survey", "hits"])
        lp = rng.choice(["", "", "f16", "bf16"])
        n, h, w = rng.randint(5, 28), _log(rng, 48, 2048), _log(rng, 48, 2048)
        speeds, angles = _log(rng, 8, 60), _log(rng, 10, 60)
        k = min(rng.choice([1, 5, 10, 20, 50, 50, 50, 64]), speeds * angles - 2)
        while n * h * w * speeds * angles > 8e10:
            h, w = max(48, h * 2 // 3), max(48, w * 2 // 3)
        kc = min(64, k + 2) if lp == "bf16" else k
        return _step("", n, h, w, speeds, angles, k, kc, lp, grid, rng.choice([5, 7, 9, 11, 15]))
    if kind == "serve":
        return dict(kind="serve", jobs=rng.randint(2, 9), shapes=rng.randint(2, 10 ** 6),
                    k=rng.choice([10, 20, 50]), lp=rng.choice(["", "f16"]))
    if kind == "threshold":
        return dict(kind="threshold", n=rng.randint(8, 22), h=_log(rng, 128, 1536),
                    w=_log(rng, 128, 1536), speeds=rng.randint(10, 25),
                    angles=rng.randint(10, 24))
    if kind == "cluster":
        return dict(kind="cluster", hits=_log(rng, 500, 4_000_000))
    if kind == "lightcurve":
        return dict(kind="lightcurve", n=rng.randint(8, 30), h=_log(rng, 48, 512),
                    w=_log(rng, 48, 512), k=rng.choice([5, 20, 50]), q=rng.choice([0.0, 0.5, 1.0]))
    if kind == "stamps":
        return dict(kind="stamps", n=rng.randint(8, 28), h=_log(rng, 256, 2048),
                    w=_log(rng, 256, 2048), cands=_log(rng, 200, 200_000),
                    radius=rng.choice([3, 5, 5, 10]))
    return dict(kind="planes", n=rng.randint(5, 20), h=_log(rng, 64, 2048), w=_log(rng, 64, 2048),
                psf=rng.choice([5, 7, 11, 11, 15, 21]), lp=rng.choice(["", "f16", "bf16"]))


def _serve_shapes(c):
    """(n, h, w, speeds, angles) of each stack of a serving batch."""
    rng = np.random.default_rng(c["shapes"])
    return [(int(rng.integers(5, 21)), int(rng.integers(60, 400)), int(rng.integers(60, 500)),
             int(rng.integers(8, 16)), 20) for _ in range(c["jobs"])]


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------

def _polar(speeds, angles):
    s, a = np.repeat(speeds, angles.size), np.tile(angles, speeds.size)
    return np.stack([s * np.cos(a), s * np.sin(a)], axis=1)


def _velocities(c):
    ns, na = c["speeds"], c["angles"]
    grid = c.get("grid", "survey")
    if grid == "box":
        return np.stack(np.meshgrid(np.linspace(-50, 50, ns), np.linspace(-50, 50, na),
                                    indexing="ij"), -1).reshape(-1, 2)
    if grid == "hits":
        return _polar(np.linspace(1.0, 5.7, ns) * 24.0 / 0.26, np.deg2rad(np.linspace(-12, 12, na)))
    return _polar(np.linspace(80.0, 400.0, ns), np.linspace(-0.5, 0.5, na))


def _times(c):
    n = c["n"]
    if c.get("grid") == "box":
        return np.arange(n) * 0.05
    gap = 1.6 / 24.0 if c.get("grid") == "hits" else 0.06
    return np.array([i // 5 + gap * (i % 5) for i in range(n)], dtype=np.float64)


def _psf(size):
    """Pixel-integrated Gaussian of unit sum, sigma 1.5 (1 below 9 x 9)."""
    sigma = 1.5 if size >= 9 else 1.0
    u = torch.arange(-(size // 2), size // 2 + 1, dtype=torch.float64)
    g = torch.special.ndtr((u + 0.5) / sigma) - torch.special.ndtr((u - 0.5) / sigma)
    p = torch.outer(g, g)
    return (p / p.sum()).to(torch.float32).numpy(), sigma


def _images(c, seed, flashes_per_16m=20000.0, sources_per_16m=100.0):
    """img, var, mask [n][h][w] on the GPU: noise, moving sources, flashes."""
    n, h, w = c["n"], c["h"], c["w"]
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    ys = torch.arange(h, device=DEV, dtype=torch.float64) / h
    xs = torch.arange(w, device=DEV, dtype=torch.float64) / w
    phase = rng.random((n, 2))
    img = torch.randn((n, h, w), generator=gen, device=DEV)
    var = torch.empty_like(img)
    for i in range(n):
        var[i] = 1.0 + 0.2 * torch.outer(torch.sin(2 * math.pi * (ys + phase[i, 1])),
                                         torch.sin(2 * math.pi * (xs + phase[i, 0])))
    img *= var
    var.square_()
    mask = (torch.rand((n, h, w), generator=gen, device=DEV) < 0.01).to(torch.uint8)
    # Point sources as (image, x, y, flux): each mover in every image, each
    # flash in one.  Flux for the wanted signal-to-noise in noise of 1.
    psf, sigma = _psf(c.get("psf", 11))
    unit = math.sqrt(float((psf.astype(np.float64) ** 2).sum()))
    ns = max(1, int(round(sources_per_16m * h * w / 4096 ** 2)))
    nf = int(round(flashes_per_16m * h * w / 4096 ** 2))
    vel, t = _velocities(c), _times(c)
    x0, y0 = rng.uniform(0, w, ns), rng.uniform(0, h, ns)
    v = vel[rng.integers(0, len(vel), ns)]
    flux = rng.uniform(5, 20, ns) / (unit * math.sqrt(n))
    src = [np.stack([np.full(ns, i), x0 + v[:, 0] * t[i], y0 + v[:, 1] * t[i], flux], 1)
           for i in range(n)]
    src.append(np.stack([rng.integers(0, n, nf), rng.uniform(0, w, nf), rng.uniform(0, h, nf),
                         rng.uniform(10, 100, nf) / unit], 1))
    s = torch.from_numpy(np.concatenate(src))
    r = int(math.ceil(5 * sigma))
    off = torch.arange(-r, r + 1, dtype=torch.float64)
    px, py = torch.floor(s[:, 1, None]) + off, torch.floor(s[:, 2, None]) + off
    cdf = torch.special.ndtr
    gx = cdf((px + 0.5 - s[:, 1, None]) / sigma) - cdf((px - 0.5 - s[:, 1, None]) / sigma)
    gy = cdf((py + 0.5 - s[:, 2, None]) / sigma) - cdf((py - 0.5 - s[:, 2, None]) / sigma)
    val = s[:, 3, None, None] * gy[:, :, None] * gx[:, None, :]
    at = ((s[:, 0, None, None] * h + py[:, :, None]) * w + px[:, None, :])
    ok = ((py >= 0) & (py < h))[:, :, None] & ((px >= 0) & (px < w))[:, None, :]
    # Overlaps are summed on the host in a fixed order; each pixel is written once.
    where, inv = np.unique(at[ok].to(torch.int64).numpy(), return_inverse=True)
    add = np.bincount(inv, weights=val[ok].numpy(), minlength=where.size).astype(np.float32)
    at = torch.from_numpy(where).to(DEV)
    flat = img.view(-1)
    flat[at] = flat[at] + torch.from_numpy(add).to(DEV)
    return img, var, mask


def _planes_of(img, var, mask, psf, dtype):
    """The likelihood planes [n][h][w][2] by plain torch in `dtype`."""
    n, h, w = img.shape
    ph, pw = psf.shape
    out = torch.empty((n, h, w, 2), dtype=dtype, device=img.device)
    taps = torch.from_numpy(psf).to(dtype)
    for i in range(n):
        ok = (mask[i] == 0) & torch.isfinite(img[i]) & torch.isfinite(var[i]) & (var[i] > 0)
        wt = torch.where(ok, 1.0 / var[i].to(dtype), 0.0)
        a = torch.where(ok, img[i].to(dtype) / var[i].to(dtype), 0.0)
        pad = (pw // 2, pw // 2, ph // 2, ph // 2)
        a, wt = torch.nn.functional.pad(a, pad), torch.nn.functional.pad(wt, pad)
        psi, phi = torch.zeros((2, h, w), dtype=dtype, device=img.device)
        for u in range(ph):
            for v in range(pw):
                tap = float(taps[u, v])
                psi += a[u:u + h, v:v + w] * tap
                phi += wt[u:u + h, v:v + w] * (tap * tap)
        out[i, :, :, 0] = torch.where(ok, psi, 0.0)
        out[i, :, :, 1] = torch.where(ok, torch.where(phi > 0, phi, -0.0), 0.0)
    return out


def _shift(vel, t):
    """[V][N][2] pixel offsets: floor(v * tau + 0.5)."""
    return np.floor(vel[:, None, :] * (t - t[0])[None, :, None] + 0.5).astype(np.int64)


def _sums(planes, off):
    """Psi, Phi [h][w] of one velocity (offsets [n][2]) from every start pixel."""
    n, h, w, _ = planes.shape
    s = torch.zeros((h, w, 2), dtype=planes.dtype, device=planes.device)
    for i in range(n):
        dx, dy = int(off[i, 0]), int(off[i, 1])
        ya, yb, xa, xb = max(0, -dy), min(h, h - dy), max(0, -dx), min(w, w - dx)
        if ya < yb and xa < xb:
            s[ya:yb, xa:xb] += planes[i, ya + dy:yb + dy, xa + dx:xb + dx]
    return s[..., 0], s[..., 1]


def _topk_of(planes, t, vel, k):
    """(nu, alpha, velocity index) [h][w][k], best first, by plain torch."""
    n, h, w, _ = planes.shape
    off = _shift(vel, t)
    best = None
    for j0 in range(0, len(vel), 64):
        js = range(j0, min(len(vel), j0 + 64))
        nu = torch.empty((h * w, len(js)), dtype=planes.dtype, device=planes.device)
        al = torch.empty_like(nu)
        for q, j in enumerate(js):
            p, f = _sums(planes, off[j])
            nu[:, q] = torch.where(f > 0, p / f.sqrt(), -math.inf).reshape(-1)
            al[:, q] = torch.where(f > 0, p / f, 0.0).reshape(-1)
        jj = torch.arange(j0, j0 + len(js), device=planes.device).expand(h * w, -1)
        if best is not None:
            nu, al, jj = (torch.cat(x, 1) for x in zip(best, (nu, al, jj)))
        top, at = torch.sort(nu, dim=1, descending=True, stable=True)
        best = top[:, :k], al.gather(1, at[:, :k]), jj.gather(1, at[:, :k])
    return tuple(x.reshape(h, w, k) for x in best)


def _hit_list(c, seed):
    """Distinct hits (y, x, j) in clumps around random centres, as an int32
    [hits][6] list, on the survey's frame and velocities; a frame smaller in
    proportion for a shorter list."""
    n, vel = c["hits"], _polar(np.linspace(80.0, 400.0, 25), np.linspace(-0.5, 0.5, 24))
    side = max(64, int(4096 * math.sqrt(n / 1e7)))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def ints(lo, hi, m):
        return torch.randint(lo, hi, (m,), generator=gen, device=DEV)
    nc, m = max(1, n // 10), int(n * 1.3) + 64
    cx, cy, cj = ints(0, side, nc), ints(0, side, nc), ints(0, len(vel), nc)
    pick = ints(0, nc, m)
    x = (cx[pick] + ints(-6, 7, m)).clamp(0, side - 1)
    y = (cy[pick] + ints(-6, 7, m)).clamp(0, side - 1)
    j = (cj[pick] + ints(-2, 3, m)).clamp(0, len(vel) - 1)
    key = torch.unique((y * side + x) * len(vel) + j)
    key = key[torch.randperm(key.numel(), generator=gen, device=DEV)[:n]]
    hits = torch.zeros((key.numel(), 6), dtype=torch.int32, device=DEV)
    hits[:, 0] = (key // len(vel)) % side
    hits[:, 1] = key // len(vel) // side
    hits[:, 2] = key % len(vel)
    u = torch.rand((2, key.numel()), generator=gen, device=DEV)
    hits[:, 3] = (10.0 - 2.0 * torch.log1p(-u).sum(0)).to(torch.float32).view(torch.int32)
    hits[:, 5] = 15
    return hits, vel


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "cluster":
        hits, vel = _hit_list(c, seed)
        n = hits.shape[0]
        ws = torch.empty(max(256, lib.load().kb_cluster_workspace_bytes(n, len(vel))),
                         dtype=torch.uint8, device=DEV)
        return dict(case=c, hits=hits, vel=vel, span=2.24, ws=ws)
    if kind == "serve":
        jobs = []
        for q, (n, h, w, ns, na) in enumerate(_serve_shapes(c)):
            cq = dict(n=n, h=h, w=w, speeds=ns, angles=na, psf=11)
            jobs.append(dict(images=_images(cq, seed * 64 + q), t=_times(cq), vel=_velocities(cq)))
        return dict(case=c, jobs=jobs, psf=_psf(11)[0])
    if kind == "stamps":
        c = dict(c, speeds=25, angles=24)
    if kind == "lightcurve":
        c = dict(c, speeds=10, angles=20)
    if kind == "planes":
        c = dict(c, speeds=2, angles=2)
    # Flashes: the bright-pixel mask's and the light-curve filter's workloads
    # are full of them; the threshold search meets a few.
    many = c.get("grid") == "hits" or kind == "lightcurve"
    img, var, mask = _images(c, seed, 20000.0 if many else 100.0 if kind == "threshold" else 0.0)
    s = dict(case=c, img=img, var=var, mask=mask, t=_times(c), vel=_velocities(c),
             psf=_psf(c.get("psf", 11))[0])
    if kind == "threshold":
        s["ws"] = lib.alloc_workspace(c["n"], c["h"], c["w"], len(s["vel"]), DEV)
        s["hits"] = lib.alloc_hits(MAX_HITS, DEV)
    if kind == "lightcurve":
        s["planes"] = _planes_of(img, var, mask, s["psf"], torch.float32)
        s["cand"] = _topk_of(s["planes"], s["t"], s["vel"], c["k"])[2].to(torch.int32).contiguous()
        s["ws"] = lib.alloc_workspace(c["n"], c["h"], c["w"], len(s["vel"]), DEV)
        del s["img"], s["var"], s["mask"]
    if kind == "stamps":
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed + 1)
        at = torch.randint(0, c["h"] * c["w"], (c["cands"],), generator=gen, device=DEV).sort()[0]
        cand = torch.zeros((c["cands"], 6), dtype=torch.int32, device=DEV)
        cand[:, 0], cand[:, 1] = at % c["w"], at // c["w"]
        cand[:, 2] = torch.randint(0, len(s["vel"]), (c["cands"],), generator=gen, device=DEV)
        s["cand"] = cand
        s["ws"] = lib.alloc_workspace(c["n"], c["h"], c["w"], len(s["vel"]), DEV)
    return s


# ---------------------------------------------------------------------------
# One pass.
# ---------------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "step":
        if c["grid"] == "hits":
            lib.mask_bright(s["img"], s["mask"], 5.0)
        return lib.run_search(s["img"], s["var"], s["mask"], s["t"], s["psf"], s["vel"], c["k"],
                              k_cand=c["kc"], lp=c["lp"] or None)
    if kind == "serve":
        jobs, f32 = [], []
        for j in s["jobs"]:
            img, var, mask = j["images"]
            n, h, w = img.shape
            d = dict(t=j["t"], vel=j["vel"], out=lib.alloc_candidates(h, w, c["k"], img.device))
            if c["lp"]:
                p, d["planes"], d["lp_scale"] = lib.make_psi_phi(img, var, mask, s["psf"],
                                                                 lp=c["lp"])
            else:
                p = d["planes"] = lib.make_psi_phi(img, var, mask, s["psf"])
            f32.append(p)
            jobs.append(d)
        lib.search_batch(jobs, c["k"])
        if c["lp"]:
            return [lib.topk(d["out"], c["k"], p.shape[0], rescore=(p, d["t"], d["vel"], None))
                    for d, p in zip(jobs, f32)]
        return [lib.topk(d["out"], c["k"], p.shape[0], out=d["out"]) for d, p in zip(jobs, f32)]
    if kind == "threshold":
        planes = lib.make_psi_phi(s["img"], s["var"], s["mask"], s["psf"])
        count = lib.search_threshold(planes, s["t"], s["vel"], NU_MIN, s["hits"],
                                     workspace=s["ws"])
        # The number of hits sizes what follows, so it is read back; the list
        # comes in no order, so it is put in one.
        found = s["hits"][:min(int(count), MAX_HITS)]
        key = (found[:, 1].to(torch.int64) * c["w"] + found[:, 0]) * len(s["vel"]) + found[:, 2]
        found = found[torch.argsort(key)]
        rep = lib.cluster_hits(found, found.shape[0], s["vel"], float(s["t"][-1] - s["t"][0]), EPS)
        out = torch.zeros((MAX_HITS, 7), dtype=torch.int32, device=found.device)
        out[:len(rep), :6], out[:len(rep), 6] = found, rep
        score = out[:, 3:5].contiguous().view(torch.float32)
        return dict(planes=planes, nu=score[:, 0], alpha=score[:, 1], at=out[:, :3],
                    nobs_rep=out[:, 5:])
    if kind == "cluster":
        return lib.cluster_hits(s["hits"], s["hits"].shape[0], s["vel"], s["span"], EPS,
                                workspace=s["ws"])
    if kind == "lightcurve":
        return lib.lightcurve_filter(s["planes"], s["t"], s["vel"], s["cand"],
                                     sigma_cut=SIGMA_CUT, q=c["q"], workspace=s["ws"],
                                     rejected=True)
    if kind == "stamps":
        return lib.stamps(s["img"], s["var"], s["mask"], s["t"], s["vel"], s["cand"], c["cands"],
                          c["radius"], *STAMP_LIMITS, workspace=s["ws"])
    return lib.make_psi_phi(s["img"], s["var"], s["mask"], s["psf"], lp=c["lp"] or None)


def _step_work(n, h, w, nv, k, psf, lp):
    pix = n * h * w
    return {"bytes": pix * (9 + 8 + (4 if lp else 0)) + 14 * h * w * k,
            "flops": pix * (4 * psf * psf + 2 * nv)}


def work(case):
    c, kind = case, case["kind"]
    if kind == "cluster":
        return {"bytes": c["hits"] * 28, "flops": 0}
    if kind == "serve":
        parts = [_step_work(n, h, w, ns * na, c["k"], 11, c["lp"])
                 for n, h, w, ns, na in _serve_shapes(c)]
        return {q: sum(p[q] for p in parts) for q in ("bytes", "flops")}
    pix = c["n"] * c["h"] * c["w"]
    if kind == "step":
        return _step_work(c["n"], c["h"], c["w"], c["speeds"] * c["angles"], c["k"], c["psf"],
                          c["lp"])
    if kind == "threshold":
        return _step_work(c["n"], c["h"], c["w"], c["speeds"] * c["angles"], 0, 11, "")
    if kind == "lightcurve":
        cands = c["h"] * c["w"] * c["k"]
        # Per observation two predictions (two divisions each) and a residual.
        return {"bytes": pix * 8 + cands * 22, "flops": cands * c["n"] * 24}
    if kind == "stamps":
        side = 2 * c["radius"] + 1
        per = side * side * c["n"]
        return {"bytes": min(pix * 9, c["cands"] * per * 9) +
                c["cands"] * (24 + side * side * 4 + 49), "flops": c["cands"] * per}
    return {"bytes": pix * (9 + 8 + (4 if c["lp"] else 0)), "flops": pix * 4 * c["psf"] ** 2}


# ---------------------------------------------------------------------------
# The same in 64 bits by plain torch.
# ---------------------------------------------------------------------------

def _exact_step(img, var, mask, t, psf, vel, k):
    planes = _planes_of(img, var, mask, psf, torch.float64)
    if planes.numel() / 2 * len(vel) > EXACT_TIE:
        return planes, (None, None, None, None)
    nu, alpha, _ = _topk_of(planes, t, vel, k)
    return planes, (nu, alpha, None, None)


def _exact_threshold(s):
    planes = _planes_of(s["img"], s["var"], s["mask"], s["psf"], torch.float64)
    off = _shift(s["vel"], s["t"])
    at, nus, als = [], [], []
    for j in range(len(s["vel"])):
        p, f = _sums(planes, off[j])
        nu = torch.where(f > 0, p / f.sqrt(), -math.inf).reshape(-1)
        hit = torch.nonzero(nu >= NU_MIN)[:, 0]
        at.append(hit * len(s["vel"]) + j)
        nus.append(nu[hit])
        als.append((p.reshape(-1)[hit] / f.reshape(-1)[hit]))
    order = torch.argsort(torch.cat(at))[:MAX_HITS]
    nu, alpha = torch.zeros((2, MAX_HITS), dtype=torch.float64, device=DEV)
    nu[:len(order)], alpha[:len(order)] = torch.cat(nus)[order], torch.cat(als)[order]
    return dict(planes=planes, nu=nu, alpha=alpha, at=None, nobs_rep=None)


def _exact_lightcurve(s):
    """The filter of one candidate after another, many candidates at a time."""
    c, planes = s["case"], s["planes"]
    n, h, w, _ = planes.shape
    off = torch.from_numpy(_shift(s["vel"], s["t"])).to(DEV)
    tau, q, c2 = (s["t"] - s["t"][0]).tolist(), c["q"], SIGMA_CUT ** 2
    outs = [[], [], []]
    rows = max(1, 4_000_000 // (w * c["k"]))
    for y0 in range(0, h, rows):
        j = s["cand"][y0:y0 + rows].to(torch.int64)
        y = torch.arange(y0, y0 + j.shape[0], device=DEV)[:, None, None] + off[j][..., 1].movedim(3, 0)
        x = torch.arange(w, device=DEV)[None, :, None] + off[j][..., 0].movedim(3, 0)
        ok = (y >= 0) & (y < h) & (x >= 0) & (x < w)
        i = torch.arange(n, device=DEV)[:, None, None, None].expand_as(y)
        v = torch.where(ok[..., None], planes[i, y.clamp(0, h - 1), x.clamp(0, w - 1)], 0.0)
        v = v.reshape(n, -1, 2)
        # Validity is in phi's bits: a valid pixel's phi is never +0.
        obs = (v[..., 1].contiguous().view(torch.int32) != 0) & ok.reshape(n, -1)
        psi, phi = v[..., 0].double(), v[..., 1].double()
        keep, todo = obs.clone(), torch.arange(psi.shape[1], device=DEV)
        while todo.numel():
            ps, ph, kp = psi[:, todo], phi[:, todo], keep[:, todo]

            def predict(order):
                J = torch.zeros_like(ps[0])
                H, tp, seen, got = J.clone(), J.clone(), kp[0] & False, {}
                for m in order:
                    d = 1.0 + q * (tp - tau[m]).abs() * J
                    d = torch.where(seen & kp[m], d, 1.0)
                    J, H = J / d, H / d
                    got[m] = J, H
                    J, H = J + torch.where(kp[m], ph[m], 0.0), H + torch.where(kp[m], ps[m], 0.0)
                    tp, seen = torch.where(kp[m], tau[m], tp), seen | kp[m]
                return got
            fwd, bwd = predict(range(n)), predict(range(n - 1, -1, -1))
            worst, at = torch.full_like(ps[0], -1.0), torch.zeros_like(todo)
            for m in range(n - 1, -1, -1):
                J, H = fwd[m][0] + bwd[m][0], fwd[m][1] + bwd[m][1]
                a, dv = ps[m] * J - ph[m] * H, (ph[m] * J) * (J + ph[m])
                r = torch.where(dv > 0, a * a / dv, 0.0)
                up = kp[m] & (r >= worst)
                worst, at = torch.where(up, r, worst), torch.where(up, m, at)
            todo, at = todo[worst > c2], at[worst > c2]
            keep[at, todo] = False
        P, F = torch.where(keep, psi, 0.0).sum(0), torch.where(keep, phi, 0.0).sum(0)
        for o, x in zip(outs, (torch.where(F > 0, P / F.sqrt(), -math.inf),
                               torch.where(F > 0, P / F, 0.0))):
            o.append(x)
    nu, al = (torch.cat(o).reshape(h, w, c["k"]) for o in outs[:2])
    return nu, al, None, None


def _exact_stamps(s):
    c = s["case"]
    n, h, w, R = c["n"], c["h"], c["w"], c["radius"]
    off = torch.from_numpy(_shift(s["vel"], s["t"])).to(DEV)
    d = torch.arange(-R, R + 1, device=DEV)
    moments, stamps = [], []
    u, v = d.double()[None, None, :], d.double()[None, :, None]
    for part in s["cand"].to(torch.int64).split(32768):
        acc, cnt = (torch.zeros((len(part), 2 * R + 1, 2 * R + 1), dtype=torch.float64, device=DEV)
                    for _ in range(2))
        for i in range(n):
            o = off[part[:, 2], i]
            y = (part[:, 1] + o[:, 1])[:, None, None] + d[None, :, None]
            x = (part[:, 0] + o[:, 0])[:, None, None] + d[None, None, :]
            ok = (y >= 0) & (y < h) & (x >= 0) & (x < w)
            y, x = torch.broadcast_tensors(y.clamp(0, h - 1), x.clamp(0, w - 1))
            im, va = s["img"][i, y, x], s["var"][i, y, x]
            ok = ok & (s["mask"][i, y, x] == 0) & torch.isfinite(im) & torch.isfinite(va) & (va > 0)
            acc += torch.where(ok, im.double(), 0.0)
            cnt += ok
        S = torch.where(cnt > 0, acc / cnt, 0.0)

        def m(wt):
            return (wt * S).sum((1, 2))
        m00 = m(1.0)
        ub, vb = m(u) / m00, m(v) / m00
        moments.append(torch.stack([m00, ub, vb, m(u * u) / m00 - ub * ub,
                                    m(v * v) / m00 - vb * vb, m(u * v) / m00 - ub * vb], 1))
        stamps.append(S)
    return None, torch.cat(moments), torch.cat(stamps)


def exact(case, seed):
    if case["kind"] == "cluster":
        return None
    s = prepare(case, seed)
    c, kind = s["case"], s["case"]["kind"]
    if kind == "serve":
        return [_exact_step(*j["images"], j["t"], s["psf"], j["vel"], c["k"])[1]
                for j in s["jobs"]]
    if kind == "threshold":
        return _exact_threshold(s)
    if kind == "lightcurve":
        return _exact_lightcurve(s)
    if kind == "stamps":
        return _exact_stamps(s)
    if kind == "planes":
        planes = _planes_of(s["img"], s["var"], s["mask"], s["psf"], torch.float64)
        return (planes, None, None) if c["lp"] else planes
    mask = s["mask"]
    if c["grid"] == "hits":
        mask = mask | (s["img"] > 5.0).to(torch.uint8)
    return _exact_step(s["img"], s["var"], mask, s["t"], s["psf"], s["vel"], c["k"])
