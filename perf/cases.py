"""Workloads whose speed matters to a user of this package, each one pass through its public entry points.

Every case is a dict of plain values with a ``kind``:

* ``overlay``      the whole avalanche overlay of one DEM (normals -> release map -> trajectories);
* ``pass``         normals and release map in one call, then the trajectory pass (the benchmark's step);
* ``trajectories`` the trajectory pass alone, DEM and release map already there (a moved parameter slider);
* ``sweep``        a batched ensemble: tiles x scenarios crossed with friction parameter sets;
* ``gradient``     one calibration gradient: smooth deposit, mean squared error, adjoint (autograd);
* ``smooth``       the smooth forward with the velocity raster;
* ``calibrate``    some Adam iterations on (mu, xi);
* ``fine``         release texture finer than the DEM: normals, fine release map, trajectories with the
                   runout-angle stop;
* ``snow``         normals and the snow-cover overlay;
* ``mipmap``       the mipmap of a count and a speed raster.

Terrain is seeded fractal noise of the two shapes the benchmark uses: an incline that runs out onto a flat
(long paths, some 130 steps) and ridged alpine relief (rough at the cell scale, paths of some 7 to 17 steps).
"""
import math

import numpy as np
import torch

import paper_2506_23364_amd as avl

DEV = "cuda"
G2 = 2.0 * 9.81
INF = float("inf")

# mean accepted steps of a particle, measured with the parameters below (for work())
MEAN_STEPS = {"incline": 130.0, "alpine": 12.0}
STEP_FLOPS = 130.0  # binary32 operations of one particle step (direction, move, bilinear patch, energy, random numbers)


def listed():
    return [
        # The smallest whole overlay: 501 x 151 texels (the size of the paper's small data set), recomputed while
        # the user drags a slider. Launches and latency count.
        dict(name="overlay_small", kind="overlay", terrain="alpine", H=501, W=151, cell=5.0, P=4, S=1000, q=0.7,
             mu=0.25, xi=1500.0),
        # One trajectory pass over a 256^2 slope with long paths (the benchmark's small workload).
        dict(name="trajectories_slope", kind="trajectories", terrain="incline", H=256, W=256, cell=10.0, P=16, S=2000,
             q=0.7, mu=0.25, xi=1500.0, alpha=-1.0),
        # The overlay of a 2048^2 alpine tile with 256 particles per release texel (the benchmark's alpine tile).
        dict(name="overlay_alpine", kind="overlay", terrain="alpine", H=2048, W=2048, cell=10.0, P=256, S=4000, q=0.93,
             mu=0.2, xi=2000.0),
        # The benchmark's headline: a whole region of 8192^2 texels at 5 m.
        dict(name="pass_region", kind="pass", terrain="alpine", H=8192, W=8192, cell=5.0, P=64, S=8000, q=0.7,
             mu=0.2, xi=2000.0),
        # An interactive parameter sweep over a few small odd-sized tiles.
        dict(name="sweep_small", kind="sweep", H=243, W=250, cell=10.0, tiles=4, params=8, cells=300, P=16, S=1000),
        # An ensemble: 8 tiles of 1024^2, one scenario each, 32 parameter sets (a quarter of the benchmark's).
        dict(name="sweep_ensemble", kind="sweep", H=1024, W=1024, cell=10.0, tiles=8, params=32, cells=6000, P=32,
             S=2000),
        # One gradient of the benchmark's calibration scene.
        dict(name="gradient_scene", kind="gradient", terrain="alpine", H=1024, W=1024, cell=10.0, cells=5000, P=128,
             S=3000, mu=0.26, xi=1400.0),
        # The smooth forward with both rasters on long paths (checkpoints, velocity splats at every step).
        dict(name="smooth_slope", kind="smooth", terrain="incline", H=256, W=256, cell=10.0, cells=4000, P=16, S=2000,
             mu=0.25, xi=1500.0),
        # A short calibration run on an odd-sized tile.
        dict(name="calibrate_tile", kind="calibrate", terrain="alpine", H=501, W=640, cell=10.0, cells=1500, P=64,
             S=2000, mu=0.26, xi=1400.0, iters=20),
        # Release points at 2 x 2 texels per DEM cell, with the runout-angle stop.
        dict(name="fine_release", kind="fine", terrain="alpine", H=1001, W=1203, cell=10.0, mult=2, P=32, S=2000,
             q=0.9, mu=0.2, xi=2000.0, alpha=22.0),
        # The snow overlay of a large odd-sized region: two streaming passes.
        dict(name="snow_region", kind="snow", terrain="alpine", H=3000, W=5001, cell=5.0),
        # The multi-resolution overlay of a whole region's rasters.
        dict(name="mipmap_region", kind="mipmap", H=8192, W=8191),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, uniform in its logarithm (odd sizes as likely as even ones)."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _friction(rng):
    return dict(mu=round(rng.uniform(0.15, 0.35), 3), xi=round(rng.uniform(800.0, 2500.0), 1))


def draw(rng):
    kind = rng.choice(["overlay", "pass", "trajectories", "sweep", "gradient", "smooth", "calibrate", "fine", "snow",
                       "mipmap"])
    cell = rng.choice([5.0, 10.0])
    if kind in ("overlay", "pass", "trajectories"):
        terrain = rng.choice(["incline", "alpine"])
        top = 400 if terrain == "incline" else 4000
        H, W = _log(rng, 64, top), _log(rng, 64, top)
        P = min(_log(rng, 1, 256), max(1, int(4.0e8 / (0.09 * H * W * MEAN_STEPS[terrain]))))
        c = dict(kind=kind, terrain=terrain, H=H, W=W, cell=cell, P=P, S=_log(rng, 200, 8000),
                 q=round(rng.uniform(0.7, 0.95), 3), **_friction(rng))
        if kind == "trajectories":
            c["alpha"] = rng.choice([-1.0, -1.0, round(rng.uniform(18.0, 30.0), 1)])
        return c
    if kind == "sweep":
        tiles, params = _log(rng, 1, 8), _log(rng, 2, 64)
        side = int(math.sqrt(2.6e8 / (tiles * params)))  # the rasters of the listed ensemble at most
        H, W = _log(rng, 64, min(1024, side)), _log(rng, 64, min(1024, side))
        return dict(kind=kind, H=H, W=W, cell=cell, tiles=tiles, params=params, cells=min(_log(rng, 50, 6000), H * W // 8),
                    P=_log(rng, 4, 32), S=_log(rng, 500, 4000))
    if kind in ("gradient", "smooth", "calibrate"):
        terrain = rng.choice(["incline", "alpine"])
        top = 300 if terrain == "incline" else 1400
        H, W = _log(rng, 96, top), _log(rng, 96, top)
        c = dict(kind=kind, terrain=terrain, H=H, W=W, cell=cell, cells=min(_log(rng, 100, 6000), H * W // 10),
                 P=_log(rng, 8, 128) if terrain == "alpine" else _log(rng, 4, 24), S=_log(rng, 300, 3000),
                 **_friction(rng))
        if kind == "calibrate":
            c["iters"] = rng.randint(5, 30)
        return c
    if kind == "fine":
        H, W = _log(rng, 96, 1400), _log(rng, 96, 1400)
        return dict(kind=kind, terrain="alpine", H=H, W=W, cell=cell, mult=rng.choice([2, 2, 3, 4]), P=_log(rng, 1, 32),
                    S=_log(rng, 500, 4000), q=round(rng.uniform(0.85, 0.97), 3),
                    alpha=rng.choice([-1.0, round(rng.uniform(18.0, 30.0), 1)]), **_friction(rng))
    if kind == "snow":
        return dict(kind=kind, terrain="alpine", H=_log(rng, 100, 6000), W=_log(rng, 100, 6000), cell=cell)
    return dict(kind="mipmap", H=_log(rng, 100, 8192), W=_log(rng, 100, 8192))


# ------------------------------------------------------------------------------------------------ inputs


def _generator(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _fractal(size, gen, hurst=0.8):
    """Diamond-square fractional noise on a (2^k + 1)^2 grid that covers `size`."""
    levels = max(1, math.ceil(math.log2(max(size, 2))))
    n = 1 << levels
    noise = lambda *s: torch.randn(*s, device=DEV, generator=gen)  # noqa: E731
    z = torch.zeros(n + 1, n + 1, device=DEV)
    z[::n, ::n] = noise(2, 2)
    step, sigma = n, 1.0
    while step > 1:
        half, sigma = step // 2, sigma * 2.0 ** -hurst
        p = z[::step, ::step]
        mid = 0.25 * (p[:-1, :-1] + p[1:, :-1] + p[:-1, 1:] + p[1:, 1:])
        mid = mid + sigma * noise(*mid.shape)
        z[half::step, half::step] = mid
        for t, m in ((z, mid), (z.T, mid.T)):  # the edge midpoints along the rows, then along the columns
            p = t[::step, ::step]
            e = p[:, :-1] + p[:, 1:]
            e[1:] += m
            e[:-1] += m
            e[1:-1] *= 0.25
            e[0] /= 3.0
            e[-1] /= 3.0
            t[::step, half::step] = e + sigma * noise(*e.shape)
        step = half
    return z


def _dem(terrain, H, W, cell, gen):
    z = _fractal(max(H, W), gen)[:H, :W]
    if terrain == "incline":  # 35 degrees down to row 0.6 H, a quadratic fillet, then flat; 5 m of noise
        k, mid, f = math.tan(math.radians(35.0)) * cell, 0.625 * H, H / 32.0
        r = torch.arange(H, device=DEV, dtype=torch.float32)[:, None]
        base = torch.where(r <= mid - f, k * (mid - r),
                           torch.where(r < mid + f, k * (mid + f - r) ** 2 / (4.0 * f), torch.zeros_like(r)))
        z = z - z.mean()
        return (base + z * (5.0 / z.abs().max())).contiguous()
    # ridges: the folded noise, scaled to the mean steepness of the benchmark's tiles (height difference of row
    # neighbours over their distance: 0.42 on the alpine tile, 0.25 on the 8192^2 region)
    z = 2.0 * (z - z.min()) / (z.max() - z.min()) - 1.0
    z = 1.0 - z.abs()
    rough = float((z[:, 1:] - z[:, :-1]).abs().mean()) / cell
    return ((z - z.min()) * ((0.25 if max(H, W) > 4096 else 0.42) / rough)).contiguous()


def _quantile(z, q):
    return float(z.flatten().sort().values[min(int(q * z.numel()), z.numel() - 1)])


def _gradient(z, cell):
    """Central differences, one-sided at the edges."""
    gx, gy = torch.empty_like(z), torch.empty_like(z)
    for g, t in ((gx, z), (gy.T, z.T)):
        g[:, 1:-1] = (t[:, 2:] - t[:, :-2]) / (2.0 * cell)
        g[:, 0] = (t[:, 1] - t[:, 0]) / cell
        g[:, -1] = (t[:, -1] - t[:, -2]) / cell
    return gx, gy


def _steep(z, cell, zmin=-INF):
    gx, gy = _gradient(z, cell)
    s = torch.rad2deg(torch.atan(torch.hypot(gx, gy)))
    return (s >= 30.0) & (s <= 45.0) & (z >= zmin)


def _scenario(z, cell, n, gen):
    """A release area: the n texels nearest to a seeded steep texel of the upper half, steep ones first."""
    H, W = z.shape
    steep = _steep(z, cell)
    cand = (steep & (z >= z.median())).flatten().nonzero().flatten()
    if cand.numel() == 0:
        cand = torch.arange(H * W, device=DEV)
    start = int(cand[int(torch.randint(cand.numel(), (1,), device=DEV, generator=gen))])
    r = torch.arange(H, device=DEV, dtype=torch.float32)[:, None] - start // W
    c = torch.arange(W, device=DEV, dtype=torch.float32)[None, :] - start % W
    d = (r * r + c * c) * torch.where(steep, 1.0, 4.0)
    # ties between equal distances fall by the texel's index, so the area is the same on every run
    order = (d.flatten().double() * (2.0 * H * W) + torch.arange(H * W, device=DEV)).argsort()
    mask = torch.zeros(H * W, dtype=torch.uint8, device=DEV)
    mask[order[:n]] = 1
    return mask.view(H, W)


def _target(mask, n, gen):
    """An observed deposit: the released mass as a smooth blob some way off the release area."""
    H, W = mask.shape
    at = mask.nonzero().double().mean(0).tolist()
    off = (torch.rand(2, device=DEV, generator=gen) * 20.0 - 10.0).tolist()
    r = torch.arange(H, device=DEV, dtype=torch.float32)[:, None] - (at[0] + off[0])
    c = torch.arange(W, device=DEV, dtype=torch.float32)[None, :] - (at[1] + off[1])
    s = 0.5 * math.sqrt(n)
    return (n / (2.0 * math.pi * s * s) * torch.exp(-(r * r + c * c) / (2.0 * s * s))).contiguous()


def _inputs(case, seed):
    """The arrays of a case, made from the seed alone."""
    k, gen, cell = case["kind"], _generator(seed), case.get("cell", 10.0)
    H, W = case["H"], case["W"]
    if k == "mipmap":
        # about a fifth of the texels visited, few often
        hit = torch.rand(H, W, device=DEV, generator=gen) < 0.2
        counts = torch.where(hit, torch.exp(6.0 * torch.rand(H, W, device=DEV, generator=gen)).to(torch.int32), 0)
        vmax = torch.where(hit, 40.0 * torch.rand(H, W, device=DEV, generator=gen), 0.0)
        return dict(counts=counts.view(torch.uint32), vmax=vmax)
    if k == "sweep":
        dems = torch.stack([_dem("alpine", H, W, cell, _generator(seed, 1 + t)) for t in range(case["tiles"])])
        masks, most = [], case["cells"]
        for t in range(case["tiles"]):  # scenarios of different sizes, the largest first
            masks.append(_scenario(dems[t], cell, max(1, int(most * (1.0 + t) ** -0.7)), gen))
        u = torch.rand(case["params"], 3, device=DEV, generator=gen).tolist()
        params = [dict(mu=0.1 + 0.3 * a, xi=500.0 + 2500.0 * b, flow_height=0.5 + 2.5 * c) for a, b, c in u]
        return dict(dem=dems, mask=torch.stack(masks), params=params)
    z = _dem(case["terrain"], H, W, cell, gen)
    s = dict(dem=z)
    if "q" in case:
        s["zmin"] = _quantile(z, case["q"])
    if k == "trajectories":
        s["mask"] = _steep(z, cell, s["zmin"]).to(torch.uint8)
    if k in ("gradient", "smooth", "calibrate"):
        n = case["cells"]
        s["mask"] = _scenario(z, cell, n, gen)
        s["mass"] = (0.5 + torch.rand(H, W, device=DEV, generator=gen)) * s["mask"]
        s["target"] = _target(s["mask"], n, gen)
    if k == "snow":
        s["line"] = _quantile(z, 0.4)
    return s


def _tan_alpha(case):
    a = case.get("alpha", -1.0)
    return math.tan(math.radians(a)) if a >= 0.0 else -1.0


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], s["seed"] = case, int(seed) + 1
    if case["kind"] == "sweep":
        # every tile's scenario with every parameter set, parameters and run table on the device
        s["runs"] = avl.runs_tensor([(t, t, p, t * case["params"] + p, s["seed"]) for t in range(case["tiles"])
                                     for p in range(case["params"])], DEV)
        s["ptab"] = avl.params_tensor(s["params"], DEV)
        n = case["tiles"] * case["params"]
        H, W = case["H"], case["W"]
        s["out"] = avl.BatchResult(torch.empty((n, H, W), dtype=torch.uint32, device=DEV),
                                   torch.empty((n, H, W), dtype=torch.float32, device=DEV),
                                   torch.empty((n, 4), dtype=torch.uint64, device=DEV),
                                   torch.empty(n, dtype=torch.int32, device=DEV))
    elif "mu" in case:
        s["par"] = avl.Params.make(mu=case["mu"], xi=case["xi"], tan_alpha=_tan_alpha(case))
    if case["kind"] == "gradient":
        s["theta"] = [torch.tensor(v, requires_grad=True) for v in (case["mu"], case["xi"], 1.0)]
        s["mass"].requires_grad_(True)
    return s


# ------------------------------------------------------------------------------------------------ one pass


def _rasters(r):
    return {"counts": r.counts.view(torch.int32), "vmax": r.vmax, "stats": r.stats.view(torch.int64)}


def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "overlay":
        nrm, mask, r = avl.overlay(s["dem"], c["cell"], 30.0, 45.0, s["zmin"], INF, s["par"], c["P"], c["S"], s["seed"])
        return {"normals": nrm, "mask": mask, **_rasters(r)}
    if k == "pass":
        nrm, mask = avl.normals_release_mask(s["dem"], c["cell"], 30.0, 45.0, s["zmin"], INF)
        r = avl.trajectories(s["dem"], mask, c["cell"], s["par"], c["P"], c["S"], s["seed"])
        return {"normals": nrm, "mask": mask, **_rasters(r)}
    if k == "trajectories":
        return _rasters(avl.trajectories(s["dem"], s["mask"], c["cell"], s["par"], c["P"], c["S"], s["seed"]))
    if k == "sweep":
        r = avl.trajectories_batched(s["dem"], s["mask"], c["cell"], s["ptab"], s["runs"], c["P"], c["S"], out=s["out"])
        return {**_rasters(r), "status": r.status}
    if k == "gradient":
        dep = avl.smooth_deposit(*s["theta"], s["mass"], s["dem"], s["mask"], c["cell"], c["P"], c["S"], s["seed"],
                                 max_release_cells=c["cells"])
        loss = ((dep - s["target"]) ** 2).mean()
        g = torch.autograd.grad(loss, [*s["theta"], s["mass"]])
        return {"deposit": dep.detach(), "mu": g[0], "xi": g[1], "h": g[2], "mass": g[3]}
    if k == "smooth":
        r = avl.trajectories_smooth(s["dem"], s["mask"], c["cell"], s["par"], c["P"], c["S"], s["seed"], mass=s["mass"],
                                    velocity=True, max_release_cells=c["cells"])
        return {"deposit": r.deposit, "deposit_q": r.deposit_q, "velocity": r.velocity, "velocity_q": r.velocity_q,
                "stats": r.stats.view(torch.int64)}
    if k == "calibrate":
        hist, p = avl.calibrate(s["dem"], s["mask"], c["cell"], s["par"], c["P"], c["S"], s["seed"], s["target"],
                                c["iters"], mass=s["mass"], max_release_cells=c["cells"])
        return {"history": hist, "mu": float(p.mu), "xi": float(p.xi)}
    if k == "fine":
        nrm = avl.normals(s["dem"], c["cell"])
        mask = avl.release_mask_fine(nrm, s["dem"], c["mult"], 30.0, 45.0, s["zmin"])
        r = avl.trajectories_fine(s["dem"], mask, c["mult"], c["cell"], s["par"], c["P"], c["S"], s["seed"])
        return {"normals": nrm, "mask": mask, **_rasters(r)}
    if k == "snow":
        nrm = avl.normals(s["dem"], c["cell"])
        return {"normals": nrm, "alpha": avl.snow_cover(nrm, s["dem"], s["line"], 200.0, 55.0, 15.0)}
    levels = avl.overlay_mipmap(s["counts"], s["vmax"])
    return [(a.view(torch.int64), b) for a, b in levels]


# ------------------------------------------------------------------------------------------------ work


def _particles(c):
    n = c["H"] * c["W"]
    if "cells" in c:
        return c["cells"] * c["P"]
    share = 0.25 if c["terrain"] == "incline" else (0.33 if max(c["H"], c["W"]) <= 4096 else 0.07)
    return share * (1.0 - c["q"]) * n * c.get("mult", 1) ** 2 * c["P"]


def work(case):
    """Bytes: each input raster read once, each output written once. Operations: the particle steps (expected number)."""
    c = case
    n = float(c["H"] * c["W"])
    k = c["kind"]
    if k == "mipmap":
        return {"bytes": n * 8.0 + n / 3.0 * 12.0, "flops": n * 8.0 / 3.0}
    if k == "snow":
        return {"bytes": n * (4.0 + 16.0 + 4.0), "flops": n * 40.0}
    if k == "sweep":
        cells = sum(max(1, int(c["cells"] * (1.0 + t) ** -0.7)) for t in range(c["tiles"]))
        return {"bytes": c["tiles"] * n * 5.0 + c["tiles"] * c["params"] * n * 8.0,
                "flops": cells * c["params"] * c["P"] * MEAN_STEPS["alpine"] * STEP_FLOPS}
    steps = _particles(c) * MEAN_STEPS[c["terrain"]]
    if k in ("overlay", "pass", "fine"):
        m = float(c.get("mult", 1) ** 2)
        return {"bytes": n * (4.0 + 16.0 + m + 8.0), "flops": n * 40.0 + steps * STEP_FLOPS}
    if k == "trajectories":
        return {"bytes": n * (4.0 + 1.0 + 8.0), "flops": steps * STEP_FLOPS}
    if k == "smooth":
        return {"bytes": n * (4.0 + 1.0 + 4.0 + 24.0), "flops": steps * (STEP_FLOPS + 20.0)}
    times = float(c.get("iters", 1))  # forward and adjoint
    return {"bytes": n * 9.0 + times * n * 16.0, "flops": times * steps * 2.2 * STEP_FLOPS}


# ------------------------------------------------------------------------------------------------ 64 bits


def _normals64(dem, cell):
    z = dem.double()
    gx, gy = _gradient(z, cell)
    n = torch.sqrt(gx * gx + gy * gy + 1.0)
    return torch.stack([-gx / n, -gy / n, 1.0 / n, torch.rad2deg(torch.atan(torch.hypot(gx, gy)))], 2)


def _window(nz, z, zmin):
    f = lambda d: float(np.float32(math.cos(math.radians(d))))  # noqa: E731
    return (nz >= f(45.0)) & (nz <= f(30.0)) & (z >= zmin)


def _lerp_rows(t, H, mult):
    """Rows of `t` filtered linearly at mult texel centres per row, clamped at the edges."""
    y = (torch.arange(H * mult, device=DEV, dtype=torch.float64) + 0.5) / mult - 0.5
    r = y.floor()
    a, b = r.long().clamp(0, H - 1), (r.long() + 1).clamp(0, H - 1)
    return t[a] + (y - r)[:, None] * (t[b] - t[a])


def _philox(n, rep, cell, run, seed):
    """Philox4x32-10 (Salmon et al. 2011): the four 32-bit words of the counter (n, rep, cell, run)."""
    m32 = 0xFFFFFFFF
    c = [n, rep, cell, torch.full_like(n, run)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p, q = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((q >> 32) & m32) ^ c[1] ^ k0, q & m32, ((p >> 32) & m32) ^ c[3] ^ k1, p & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c


def _patch(dem, x, y):
    """Corner indices and weights of the bilinear patch at (x, y), indices clamped to the grid."""
    H, W = dem.shape
    fc, fr = (x - 0.5).floor(), (y - 0.5).floor()
    ca, ra = fc.long(), fr.long()
    cb, rb = (ca + 1).clamp(0, W - 1), (ra + 1).clamp(0, H - 1)
    ca, ra = ca.clamp(0, W - 1), ra.clamp(0, H - 1)
    return (ra * W + ca, ra * W + cb, rb * W + ca, rb * W + cb), x - 0.5 - fc, y - 0.5 - fr


def _sample(dem, x, y):
    at, fx, fy = _patch(dem, x, y)
    a, b, c, d = (dem.flatten()[i] for i in at)
    top, bot = a + fx * (b - a), c + fx * (d - c)
    return top + fy * (bot - top), (b - a) + fy * ((d - c) - (b - a)), bot - top


def _splat(q, at, fx, fy, val):
    for i, w in zip(at, ((1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy)):
        q.index_add_(0, i, val * w)


def _walk(dem, texels, mult, cell, mu, xi, h, alpha, P, S, seed, run_id=0, mass=None, vmax=None, dep=None, vel=None):
    """The trajectory model in binary64 over the release texels. Fills vmax (largest speed per cell), or dep and
    vel (the smooth variant's rasters); with dep also returns the resting points and their derivatives."""
    H, W = dem.shape
    f32 = lambda v: float(np.float32(v))  # noqa: E731
    mu, xi, h, cell, per, rnd = f32(mu), f32(xi), f32(h), f32(cell), f32(0.9), f32(0.16)
    ta, cd, dl = f32(alpha) * cell, G2 / (xi * h), cell
    tex = texels.repeat_interleave(P)
    s = {"id": torch.arange(tex.numel(), device=DEV), "tex": tex, "rep": torch.arange(P, device=DEV).repeat(texels.numel())}
    s["x"], s["y"] = ((tex % (W * mult)).double() + 0.5) / mult, ((tex // (W * mult)).double() + 0.5) / mult
    s["z"], s["gx"], s["gy"] = _sample(dem, s["x"], s["y"])
    g = torch.hypot(s["gx"], s["gy"])
    inv = torch.where(g > 0, 1.0 / g, 0.0)
    s["dx"], s["dy"], s["v2"] = -s["gx"] * inv, -s["gy"] * inv, torch.zeros_like(g)
    if ta >= 0:
        s["x0"], s["y0"], s["z0"] = s["x"], s["y"], s["z"]
    if dep is not None:
        s["m"] = mass.flatten()[tex].double() / P
        for t in ("tmu", "txi", "th"):
            s[t] = torch.zeros_like(g)
    rest = []

    def end(e, t, x1, y1, tang):
        x, y = e["x"] + t * (x1 - e["x"]), e["y"] + t * (y1 - e["y"])
        at, fx, fy = _patch(dem, x, y)
        _splat(dep, at, fx, fy, e["m"])
        rest.append((e["tex"], at, fx, fy, e["m"], x1 - e["x"], y1 - e["y"], tang))

    for n in range(S):
        if s["id"].numel() == 0:
            break
        if n % 2 == 0:
            w = _philox(torch.full_like(s["id"], n // 2), s["rep"], s["tex"], run_id, seed)
            s["sx"], s["sy"] = w[2], w[3]
            ux, uy = w[0], w[1]
        else:
            ux, uy = s["sx"], s["sy"]
        unit = lambda u: (u >> 8).double() * 2.0 ** -23 - 1.0  # noqa: E731
        g = torch.hypot(s["gx"], s["gy"])
        t = torch.where(g > 0, (1.0 - per) / g, 0.0)
        wx = per * s["dx"] - t * s["gx"] + rnd * unit(ux)
        wy = per * s["dy"] - t * s["gy"] + rnd * unit(uy)
        l = torch.hypot(wx, wy)
        dx, dy = torch.where(l > 0, wx / l, s["dx"]), torch.where(l > 0, wy / l, s["dy"])
        x1, y1 = s["x"] + dx, s["y"] + dy
        inb = (x1 >= 0) & (x1 < W) & (y1 >= 0) & (y1 < H)
        z1, gx1, gy1 = _sample(dem, x1, y1)
        dz = s["z"] - z1
        num = s["v2"] + G2 * (dz - mu * dl)
        a = cd * torch.sqrt(dl * dl + dz * dz)
        stop = num <= 0
        ang = torch.zeros_like(stop)
        if ta >= 0:
            ang = ~stop & ((s["z0"] - z1) < ta * torch.hypot(x1 - s["x0"], y1 - s["y0"]))
        if dep is not None:
            i = (inb & stop).nonzero().flatten()
            e = {q: v[i] for q, v in s.items()}
            d = e["v2"] - num[i]
            t = torch.where(e["v2"] > 0, e["v2"] / d, 0.0)
            # t = v^2 / (v^2 - num), and v^2 - num depends on mu alone (it is -g2 (dz - mu dl))
            tang = [torch.where(d > 0, e["tmu"] / d - e["v2"] / (d * d) * (G2 * dl), 0.0),
                    torch.where(d > 0, e["txi"] / d, 0.0), torch.where(d > 0, e["th"] / d, 0.0)]
            end(e, t, x1[i], y1[i], tang)
            op = 1.0 + a
            s["tmu"] = (s["tmu"] - G2 * dl) / op
            s["txi"] = s["txi"] / op + num * (a / xi) / (op * op)
            s["th"] = s["th"] / op + num * (a / h) / (op * op)
        s.update(x=x1, y=y1, z=z1, gx=gx1, gy=gy1, dx=dx, dy=dy, v2=num / (1.0 + a))
        acc = (inb & ~stop & ~ang).nonzero().flatten()
        s = {q: v[acc] for q, v in s.items()}
        if vmax is not None:
            vmax.scatter_reduce_(0, s["y"].long() * W + s["x"].long(), s["v2"].sqrt(), "amax")
        if vel is not None:
            _splat(vel, *_patch(dem, s["x"], s["y"]), s["m"] * s["v2"].sqrt())
    if dep is not None and s["id"].numel():
        zero = torch.zeros_like(s["x"])
        end(s, 0.0, s["x"], s["y"], [zero, zero, zero])
    return rest


def exact(case, seed):
    """Binary64 values of the floating outputs. Whole numbers (maps, counts, statistics, fixed point rasters) have
    none: a particle whose binary64 path crosses a texel edge a rounding earlier enters another cell. A
    calibration's iterates have none either, each pass starting from the one before it, nor has a sweep of
    hundreds of runs within the time there is."""
    c, k = case, case["kind"]
    if k == "calibrate" or (k == "sweep" and c["tiles"] * c["params"] > 32):
        return None
    s = _inputs(case, seed)
    H, W = c["H"], c["W"]
    rid = int(seed) + 1
    if k == "mipmap":
        out, v = [], s["vmax"].double()
        while v.shape[0] > 1 or v.shape[1] > 1:
            v = torch.nn.functional.pad(v, (0, v.shape[1] % 2, 0, v.shape[0] % 2))
            v = torch.maximum(torch.maximum(v[::2, ::2], v[1::2, ::2]), torch.maximum(v[::2, 1::2], v[1::2, 1::2]))
            out.append((None, v))
        return out
    if k == "sweep":
        n = c["tiles"] * c["params"]
        vmax = torch.zeros(n, H * W, device=DEV, dtype=torch.float64)
        for t in range(c["tiles"]):
            tex = s["mask"][t].flatten().nonzero().flatten()
            for p, q in enumerate(s["params"]):
                r = t * c["params"] + p
                _walk(s["dem"][t].double(), tex, 1, c["cell"], q["mu"], q["xi"], q["flow_height"], -1.0, c["P"], c["S"],
                      rid, r, vmax=vmax[r])
        return {"counts": None, "vmax": vmax.view(n, H, W), "stats": None, "status": None}
    z = s["dem"].double()
    out = {}
    if k in ("overlay", "pass", "fine", "snow"):
        nrm = _normals64(s["dem"], c["cell"])
        out["normals"] = nrm
    if k == "snow":
        ramp = lambda v, lo, hi: ((v - lo) / (hi - lo)).clamp(0.0, 1.0)  # noqa: E731
        lo, hi = math.cos(math.radians(55.0)), math.cos(math.radians(40.0))
        out["alpha"] = ramp(z, s["line"], s["line"] + 200.0) * ramp(nrm[:, :, 2], lo, hi)
        return out
    if k in ("overlay", "pass", "fine", "trajectories"):
        m = c.get("mult", 1)
        if k == "trajectories":
            mask = s["mask"].bool()
        elif m == 1:
            mask = _window(nrm[:, :, 2], z, s["zmin"])
        else:
            fine = [_lerp_rows(_lerp_rows(t, H, m).T, W, m).T for t in (nrm[:, :, 2], z)]
            mask = _window(*fine, s["zmin"])
        vmax = torch.zeros(H * W, device=DEV, dtype=torch.float64)
        _walk(z, mask.flatten().nonzero().flatten(), m, c["cell"], c["mu"], c["xi"], 1.0, _tan_alpha(c), c["P"], c["S"],
              rid, vmax=vmax)
        out.update(mask=None, counts=None, vmax=vmax.view(H, W), stats=None)
        if k == "trajectories":
            del out["mask"]
        return out
    dep = torch.zeros(H * W, device=DEV, dtype=torch.float64)
    vel = torch.zeros_like(dep) if k == "smooth" else None
    tex = s["mask"].flatten().nonzero().flatten()
    rest = _walk(z, tex, 1, c["cell"], c["mu"], c["xi"], 1.0, -1.0, c["P"], c["S"], rid, mass=s["mass"], dep=dep, vel=vel)
    if k == "smooth":
        return {"deposit": dep.view(H, W), "deposit_q": None, "velocity": vel.view(H, W), "velocity_q": None,
                "stats": None}
    gd = 2.0 / (H * W) * (dep - s["target"].double().flatten())
    grad, gm = [0.0, 0.0, 0.0], torch.zeros_like(dep)
    for tx, at, fx, fy, m, ex, ey, tang in rest:
        g00, g01, g10, g11 = (gd[i] for i in at)
        gt = m * (((g01 - g00) * (1 - fy) + (g11 - g10) * fy) * ex + ((g10 - g00) * (1 - fx) + (g11 - g01) * fx) * ey)
        gm.index_add_(0, tx, (g00 * (1 - fx) * (1 - fy) + g01 * fx * (1 - fy) + g10 * (1 - fx) * fy + g11 * fx * fy) / c["P"])
        grad = [g + (gt * t).sum() for g, t in zip(grad, tang)]
    return {"deposit": dep.view(H, W), "mu": grad[0], "xi": grad[1], "h": grad[2], "mass": gm.view(H, W)}
