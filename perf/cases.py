"""The work a user of this package has it do, as timed cases.

Every case draws its inputs on the GPU from a seed, keeps what such a program
keeps between calls (star arrays, output buffers, a plan where the case is
about a plan) and makes one pass through the package's public entry points.
Sizes are those of the benchmark and its workloads, and generic ones below
them: N_* from tens of stars to 1.6e7, grids from 64 to 16384 a side.

Critical curves are not among the cases: their segments come out in no
particular order.
"""
from __future__ import annotations

import math

import torch

import paper_2211_00354_amd as lf

DEV = "cuda"


def listed():
    return [
        # the smallest useful call: a few thousand stars, a preview-sized grid;
        # latency and launches
        {"name": "deflect_2e3_192x160", "kind": "deflect", "n": 2000, "nx": 192, "ny": 160,
         "p": 12, "precision": "mixed", "kappa_s": 0.1, "gamma": 0.25},
        # the small disk workload by the exact O(N_* N_x) sum, the reference
        # method that small fields are checked with
        {"name": "direct_1e3_512", "kind": "direct", "n": 1000, "nx": 512, "ny": 512},
        # the headline benchmark: 1e6 power-law stars, 8192^2 rays, plan-less
        {"name": "deflect_1e6_8192", "kind": "deflect", "n": 1_000_000, "nx": 8192, "ny": 8192,
         "p": 12, "precision": "mixed", "kappa_s": 0.2, "gamma": 0.35},
        # a plan kept by the caller, FP64 with the derivative f', on a ragged
        # grid (Jacobians, magnifications)
        {"name": "plan_2e4_dfdz_1001x777", "kind": "plan", "n": 20_000, "nx": 1001, "ny": 777,
         "p": 24},
        # scattered rays (a ray bundle, observed positions), FP64, plan-less
        {"name": "rays_1e5_3e5_fp64", "kind": "rays", "n": 100_000, "n_rays": 300_000, "p": 20,
         "precision": "fp64"},
        # forward and backward: fitting lens positions and masses, clustered
        # lenses, scattered rays
        {"name": "gradient_2e5_1e6", "kind": "gradient", "clusters": 2000, "per": 100,
         "n_rays": 1_000_000, "p": 12, "precision": "mixed"},
        # the high-magnification map by inverse ray shooting: rays on a small
        # part of a wide star field, binned into pixels
        {"name": "map_5e6_16384", "kind": "map", "n": 5_000_000, "nx": 16384, "ny": 16384,
         "npix": 2000, "p": 17},
        # the same field by inverse polygon mapping
        {"name": "ipm_5e6_16384", "kind": "ipm", "n": 5_000_000, "nx": 16384, "ny": 16384,
         "npix": 2000, "p": 17},
        # a survey's batch of independent fields in one call
        {"name": "batch_64_2048", "kind": "batch", "fields": 64, "side": 2048, "npix": 512,
         "n_lo": 10_000, "n_hi": 200_000, "p": 12},
        # a particle halo: a clustered field of 1.6e7 particles
        {"name": "halo_1.6e7_4000", "kind": "halo", "n": 15_750_128, "side": 4000, "p": 12},
        # a chain of lens planes: the rays of the later planes are scattered
        {"name": "planes_3_5e4_1024", "kind": "planes", "planes": 3, "n": 50_000, "side": 1024,
         "p": 12},
        # the images of a few point sources: grid deflection, then Newton steps
        {"name": "images_1e3_512", "kind": "images", "n": 1000, "side": 512, "sources": 8, "p": 24},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["deflect", "deflect", "direct", "plan", "rays", "gradient", "map", "ipm", "batch",
                       "halo", "planes", "images"])
    if kind == "deflect":
        nx = _log_int(rng, 64, 8192)
        prec = rng.choice(["mixed", "mixed", "fp64"])
        return {"kind": kind, "n": _log_int(rng, 500, 1_000_000), "nx": nx,
                "ny": max(1, int(nx * rng.uniform(0.5, 1.0))), "p": rng.randint(8, 20), "precision": prec,
                "kappa_s": round(rng.uniform(0.0, 0.4), 3), "gamma": round(rng.uniform(0.0, 0.4), 3)}
    if kind == "direct":
        return {"kind": kind, "n": _log_int(rng, 10, 4000), "nx": _log_int(rng, 64, 1024),
                "ny": _log_int(rng, 64, 1024)}
    if kind == "plan":
        return {"kind": kind, "n": _log_int(rng, 500, 200_000), "nx": _log_int(rng, 64, 2048),
                "ny": _log_int(rng, 64, 2048), "p": rng.randint(12, 28)}
    if kind == "rays":
        return {"kind": kind, "n": _log_int(rng, 1000, 200_000), "n_rays": _log_int(rng, 100, 1_000_000),
                "p": rng.randint(10, 24), "precision": rng.choice(["mixed", "fp64"])}
    if kind == "gradient":
        return {"kind": kind, "clusters": _log_int(rng, 20, 2000), "per": rng.randint(20, 100),
                "n_rays": _log_int(rng, 10_000, 1_000_000), "p": rng.randint(10, 20),
                "precision": rng.choice(["mixed", "fp64"])}
    if kind in ("map", "ipm"):
        nx = _log_int(rng, 512, 16384)
        return {"kind": kind, "n": _log_int(rng, 10_000, 5_000_000), "nx": nx,
                "ny": int(nx * rng.uniform(0.6, 1.0)), "npix": max(64, nx // rng.randint(8, 12)),
                "p": rng.randint(12, 18)}
    if kind == "batch":
        return {"kind": kind, "fields": rng.randint(4, 64), "side": _log_int(rng, 128, 2048),
                "npix": rng.randint(64, 512), "n_lo": 1000, "n_hi": _log_int(rng, 5_000, 200_000),
                "p": rng.randint(10, 14)}
    if kind == "halo":
        return {"kind": kind, "n": _log_int(rng, 100_000, 15_750_000), "side": _log_int(rng, 256, 4000),
                "p": rng.randint(9, 13)}
    if kind == "planes":
        return {"kind": kind, "planes": rng.randint(2, 4), "n": _log_int(rng, 1000, 100_000),
                "side": _log_int(rng, 64, 1024), "p": rng.randint(10, 14)}
    return {"kind": kind, "n": _log_int(rng, 50, 1000), "side": _log_int(rng, 64, 512),
            "sources": rng.randint(1, 8), "p": rng.randint(20, 28)}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _disk(g, n, radius):
    """Points uniform in a disk (the star fields of the paper's Section 2.3)."""
    r = radius * torch.sqrt(_rand(g, n))
    th = (2.0 * math.pi) * _rand(g, n)
    return torch.stack([r * torch.cos(th), r * torch.sin(th)], 1).contiguous()


def _powerlaw(g, n):
    """Masses dN/dm ~ m^-2.35 on [0.1, 1], scaled to a mean of 1."""
    a = -1.35
    m = (0.1 ** a + _rand(g, n) * (1.0 - 0.1 ** a)) ** (1.0 / a)
    return m * (n / float(m.sum()))


def _grid(width, height, nx, ny):
    """A grid centred on the origin, spacings snapped to multiples of 2^-20."""
    dx, dy = (round(v * (1 << 20)) / (1 << 20) for v in (width / nx, height / ny))
    return lf.Grid(-0.5 * nx * dx, -0.5 * ny * dy, dx, dy, nx, ny)


def _halo(g, n):
    """A synthetic galaxy halo's particles: dark matter (surface density 1/r,
    axis ratio 0.75), cored gas, an exponential stellar disk and 128 central
    black holes, rotated by 30 degrees."""
    n_bh = 128
    n_dm = int(0.686 * n)
    n_gas = int(0.239 * n)
    n_st = n - n_dm - n_gas - n_bh
    R, rc, rs = 1500.0, 40.0, 6.0

    def place(r, q):
        th = (2.0 * math.pi) * _rand(g, r.numel())
        x, y = r * torch.cos(th), q * r * torch.sin(th)
        c, s = math.cos(math.pi / 6), math.sin(math.pi / 6)
        return torch.stack([c * x - s * y, s * x + c * y], 1)

    a = math.sqrt(R * R + rc * rc) - rc
    dm = place(R * _rand(g, n_dm), 0.75)
    gas = place(torch.sqrt((_rand(g, n_gas) * a + rc) ** 2 - rc * rc), 0.75)
    st = place(torch.clamp(-rs * torch.log(_rand(g, n_st) * _rand(g, n_st) + 1e-300), max=R), 0.6)
    xy = torch.cat([dm, gas, st, _randn(g, n_bh, 2)]).contiguous()
    M = 13050.0

    def full(k, v):
        return torch.full((k,), v, device=DEV, dtype=torch.float64)

    m = torch.cat([full(n_dm, 0.80 * M / n_dm), full(n_gas, 0.15 * M / n_gas),
                   full(n_st, 0.05 * M / n_st), full(n_bh, 0.03)])
    return xy, m


def _ones(n):
    return torch.ones(n, device=DEV, dtype=torch.float64)


def _out(n):
    return torch.empty((n, 2), device=DEV, dtype=torch.float64)


def prepare(case, seed):
    c, g, kind = case, _gen(seed), case["kind"]
    s = {"case": c}
    if kind == "deflect":
        # a disk of convergence 0.4, rays over its inscribed square
        m = _powerlaw(g, c["n"])
        R = math.sqrt(c["n"] / 0.4)
        side = math.sqrt(2.0) * R
        s.update(xy=_disk(g, c["n"], R), m=m, out=_out(c["nx"] * c["ny"]),
                 grid=_grid(side, side * c["ny"] / c["nx"], c["nx"], c["ny"]))
    elif kind == "direct":
        s.update(xy=_disk(g, c["n"], 26.6), m=_ones(c["n"]), out=_out(c["nx"] * c["ny"]),
                 grid=_grid(10.0, 10.0, c["nx"], c["ny"]))
    elif kind == "plan":
        R = math.sqrt(c["n"] / 0.3)
        xy, m = _disk(g, c["n"], R), _powerlaw(g, c["n"])
        grid = _grid(1.2 * R, 1.2 * R * c["ny"] / max(c["nx"], c["ny"]), c["nx"], c["ny"])
        s.update(xy=xy, m=m, grid=grid, out=_out(c["nx"] * c["ny"]), dout=_out(c["nx"] * c["ny"]),
                 plan=lf.Plan(xy, m, kappa_s=0.1, gamma=0.2, grid=grid, precision="fp64", p=c["p"]))
    elif kind == "rays":
        R = math.sqrt(c["n"] / 0.4)
        s.update(xy=_disk(g, c["n"], R), m=_powerlaw(g, c["n"]), rays=_disk(g, c["n_rays"], 0.8 * R),
                 out=_out(c["n_rays"]))
    elif kind == "gradient":
        # Gaussian clusters (sigma 0.5) in a disk of radius 60, as many rays
        # as constraints, the loss gradient at each
        n = c["clusters"] * c["per"]
        xy = torch.repeat_interleave(_disk(g, c["clusters"], 60.0), c["per"], 0) + 0.5 * _randn(g, n, 2)
        s.update(xy=xy.contiguous().requires_grad_(True), m=_ones(n).requires_grad_(True),
                 rays=_disk(g, c["n_rays"], 60.0), gy=0.01 * _randn(g, c["n_rays"], 2))
    elif kind in ("map", "ipm"):
        # mu = 50: kappa_* = 0.1 in a disk of N_* stars, rays over 240 x 120
        # around its centre
        s.update(xy=_disk(g, c["n"], math.sqrt(c["n"] / 0.1)), m=_ones(c["n"]),
                 grid=lf.Grid(-120.0, -60.0, 240.0 / c["nx"], 120.0 / c["ny"], c["nx"], c["ny"]),
                 map=lf.MapDesc(-10.0, -10.0, 20.0, c["npix"]),
                 out=torch.zeros((c["npix"], c["npix"]), device=DEV,
                                 dtype=torch.int32 if kind == "map" else torch.float64))
    elif kind == "batch":
        import random
        r = random.Random(int(seed) * 1000003 + 17)
        fields, grids, maps, outs = [], [], [], []
        for _ in range(c["fields"]):
            n = _log_int(r, c["n_lo"], c["n_hi"])
            ks, gm = r.uniform(0.05, 0.6), r.uniform(0.0, 0.6)
            R = math.sqrt(n / ks)
            side = math.sqrt(2.0) * R
            fields.append((_disk(g, n, R), _ones(n), 0.0, gm))
            grids.append(_grid(side, side, c["side"], c["side"]))
            L = max(0.8 * side * min(abs(1.0 - ks - gm), abs(1.0 - ks + gm)), 0.02 * side)
            maps.append(lf.MapDesc(-0.5 * L, -0.5 * L, L, c["npix"]))
            outs.append(torch.zeros((c["npix"], c["npix"]), device=DEV, dtype=torch.int32))
        s.update(fields=fields, grids=grids, maps=maps, out=outs)
    elif kind == "halo":
        xy, m = _halo(g, c["n"])
        s.update(xy=xy, m=m, grid=_grid(90.0, 90.0, c["side"], c["side"]), out=_out(c["side"] ** 2))
    elif kind == "planes":
        k = c["planes"]
        R = math.sqrt(c["n"] / 0.15)
        s.update(planes=[(_disk(g, c["n"], R), _powerlaw(g, c["n"]), 0.05, 0.1) for _ in range(k)],
                 beta=[[(j - i) / k if i < j else 0.0 for i in range(k)] for j in range(k)],
                 grid=_grid(1.2 * R, 1.2 * R, c["side"], c["side"]), out=_out(c["side"] ** 2))
    elif kind == "images":
        R = math.sqrt(c["n"] / 0.3)
        xy, m = _disk(g, c["n"], R), _ones(c["n"])
        grid = _grid(1.2 * R, 1.2 * R, c["side"], c["side"])
        s.update(xy=xy, m=m, grid=grid, sources=(0.4 * R * (_rand(g, c["sources"], 2) - 0.5)).contiguous(),
                 plan=lf.Plan(xy, m, gamma=0.15, grid=grid, precision="fp64", p=c["p"]),
                 out=_ones(4 * c["sources"] * (c["n"] + 64)).view(-1, 4),
                 src=torch.zeros(c["sources"] * (c["n"] + 64), device=DEV, dtype=torch.int32))
    else:
        raise ValueError(kind)
    return s


# ------------------------------------------------------------------- a pass


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "deflect":
        return lf.deflect(s["xy"], s["m"], grid=s["grid"], kappa_s=c["kappa_s"], gamma=c["gamma"],
                          precision=c["precision"], p=c["p"], out=s["out"])
    if kind == "direct":
        return lf.deflect(s["xy"], s["m"], grid=s["grid"], gamma=0.3, method="direct", out=s["out"])
    if kind == "plan":
        return lf.deflect(grid=s["grid"], plan=s["plan"], kappa_s=0.1, gamma=0.2, precision="fp64",
                          p=c["p"], out=s["out"], dfdz_out=s["dout"])
    if kind == "rays":
        return lf.deflect(s["xy"], s["m"], rays=s["rays"], gamma=0.1, precision=c["precision"],
                          p=c["p"], out=s["out"])
    if kind == "gradient":
        y = lf.LensDeflect.apply(s["xy"], s["m"], s["rays"], None, 0.0, 0.0, "fmm", c["precision"], c["p"])
        gxy, gm = torch.autograd.grad(y, (s["xy"], s["m"]), s["gy"])
        return {"y": y.detach(), "grad_xy": gxy, "grad_m": gm}
    if kind in ("map", "ipm"):
        s["out"].zero_()
        kw = dict(grid=s["grid"], map=s["map"], kappa_s=0.75, gamma=0.05, precision="mixed", p=c["p"],
                  fp32_levels=-1)
        if kind == "map":
            return lf.irs_map(s["xy"], s["m"], counts=s["out"], **kw)
        return lf.ipm_map(s["xy"], s["m"], mu=s["out"], **kw)
    if kind == "batch":
        for o in s["out"]:
            o.zero_()
        return lf.irs_map_batched(s["fields"], s["grids"], s["maps"], counts=s["out"], precision="mixed",
                                  p=c["p"])
    if kind == "halo":
        return lf.deflect(s["xy"], s["m"], grid=s["grid"], gamma=0.03, precision="mixed", p=c["p"],
                          out=s["out"])
    if kind == "planes":
        return lf.deflect_multiplane(s["planes"], beta=s["beta"], grid=s["grid"], out=s["out"],
                                     precision="mixed", p=c["p"])
    img, src = lf.find_images(s["xy"], s["m"], grid=s["grid"], sources=s["sources"], gamma=0.15,
                              precision="fp64", p=c["p"], plan=s["plan"])
    # the program's table of results, one row per image, -1 past the last
    k = min(src.numel(), s["src"].numel())
    s["out"][:k] = img[:k]
    s["src"][:k] = src[:k]
    s["out"][k:] = 0.0
    s["src"][k:] = -1
    return {"images": s["out"], "src": s["src"]}


# ------------------------------------------------------- what a pass must do


def _counts(c):
    """Stars and rays of one pass."""
    k = c["kind"]
    if k in ("deflect", "direct", "plan", "map", "ipm"):
        return c["n"], c["nx"] * c["ny"]
    if k == "rays":
        return c["n"], c["n_rays"]
    if k == "gradient":
        return c["clusters"] * c["per"], c["n_rays"]
    if k == "batch":
        lo, hi = math.log(c["n_lo"]), math.log(c["n_hi"])
        mean = (c["n_hi"] - c["n_lo"]) / (hi - lo) if hi > lo else c["n_lo"]
        return int(c["fields"] * mean), c["fields"] * c["side"] ** 2
    if k == "planes":
        return c["planes"] * c["n"], c["planes"] * c["side"] ** 2
    return c["n"], c["side"] ** 2


def work(case):
    """Stars are read (24 bytes each) and results written once; a ray takes
    its local expansion (8 p operations) and the pairs (12 operations) with
    the nine stars of its neighbourhood, a star its multipole (8 p)."""
    c, k = case, case["kind"]
    n, r = _counts(c)
    if k == "direct":
        return {"bytes": 24.0 * n + 16.0 * r, "flops": 12.0 * n * r}
    flops = r * (8.0 * c["p"] + 12.0 * 9) + n * 8.0 * c["p"]
    size = 24.0 * n
    if k in ("deflect", "halo"):
        size += 16.0 * r
    elif k == "plan":
        size += 32.0 * r
        flops *= 2
    elif k == "rays":
        size += 32.0 * r
    elif k == "gradient":
        size += 48.0 * r + 24.0 * n
        flops *= 3
    elif k == "map":
        size += 4.0 * c["npix"] ** 2
    elif k == "ipm":
        size += 8.0 * c["npix"] ** 2
    elif k == "batch":
        size += 4.0 * c["fields"] * c["npix"] ** 2
    elif k == "planes":
        size += 16.0 * c["side"] ** 2
    return {"bytes": size, "flops": flops}


# ------------------------------------------------- the same in plain FP64


def _grid_rays(g):
    x = g.x0 + (torch.arange(g.nx, device=DEV, dtype=torch.float64) + 0.5) * g.dx
    y = g.y0 + (torch.arange(g.ny, device=DEV, dtype=torch.float64) + 0.5) * g.dy
    return torch.stack([x.repeat(g.ny), y.repeat_interleave(g.nx)], 1)


def _sum(xy, m, rays, derivative=False):
    """alpha (and f') of every ray by the direct sum over the stars."""
    a = torch.empty_like(rays)
    d = torch.empty_like(rays) if derivative else None
    step = max(1, (1 << 26) // max(1, xy.shape[0]))
    for k in range(0, rays.shape[0], step):
        q = rays[k:k + step]
        dx = q[:, :1] - xy[:, 0]
        dy = q[:, 1:] - xy[:, 1]
        r2 = dx * dx + dy * dy
        w = torch.where(r2 > 0, m / r2, torch.zeros_like(r2))
        a[k:k + step, 0] = (w * dx).sum(1)
        a[k:k + step, 1] = (w * dy).sum(1)
        if derivative:
            t = torch.where(r2 > 0, w / r2, torch.zeros_like(r2))
            d[k:k + step, 0] = -(t * (dx * dx - dy * dy)).sum(1)
            d[k:k + step, 1] = (2 * t * dx * dy).sum(1)
    return (a, d) if derivative else a


def _map(rays, a, kappa_s, gamma):
    c = torch.tensor([1.0 - kappa_s - gamma, 1.0 - kappa_s + gamma], device=DEV, dtype=torch.float64)
    return c * rays - a


def exact(case, seed):
    c, kind = case, case["kind"]
    n, r = _counts(c)
    pairs = float(n) * r / (c["planes"] if kind == "planes" else 1)
    if kind in ("map", "ipm", "batch", "images") or pairs > (4e10 if kind == "gradient" else 1.6e11):
        return None
    s = prepare(case, seed)
    if kind in ("deflect", "direct", "halo"):
        rays = _grid_rays(s["grid"])
        return _map(rays, _sum(s["xy"], s["m"], rays), c.get("kappa_s", 0.0),
                    {"deflect": c.get("gamma"), "direct": 0.3, "halo": 0.03}[kind])
    if kind == "plan":
        rays = _grid_rays(s["grid"])
        a, d = _sum(s["xy"], s["m"], rays, True)
        return [_map(rays, a, 0.1, 0.2), d]
    if kind == "rays":
        return _map(s["rays"], _sum(s["xy"], s["m"], s["rays"]), 0.0, 0.1)
    if kind == "gradient":
        xy, m, rays, gy = s["xy"].detach(), s["m"].detach(), s["rays"], s["gy"]
        gxy, gm = torch.empty_like(xy), torch.empty_like(m)
        step = max(1, (1 << 26) // rays.shape[0])
        for k in range(0, m.numel(), step):
            # y = x - sum m d / |d|^2, d = ray - star
            dx = rays[:, 0] - xy[k:k + step, :1]
            dy = rays[:, 1] - xy[k:k + step, 1:]
            r2 = dx * dx + dy * dy
            w = torch.where(r2 > 0, 1.0 / r2, torch.zeros_like(r2))
            dot = (dx * gy[:, 0] + dy * gy[:, 1]) * w
            gm[k:k + step] = -dot.sum(1)
            mk = m[k:k + step]
            gxy[k:k + step, 0] = mk * (w * (gy[:, 0] - 2 * dx * dot)).sum(1)
            gxy[k:k + step, 1] = mk * (w * (gy[:, 1] - 2 * dy * dot)).sum(1)
        return {"y": _map(rays, _sum(xy, m, rays), 0.0, 0.0), "grad_xy": gxy, "grad_m": gm}
    # planes: x_j = x_0 - sum_{i<j} beta_ij alpha_i, y = x_0 - sum_i alpha_i,
    # alpha_i with the plane's smooth terms; lf reads beta[j][i] for i < j
    x0 = _grid_rays(s["grid"])
    alphas = []
    for j, (xy, m, ks, gm) in enumerate(s["planes"]):
        x = x0.clone()
        for i in range(j):
            x -= s["beta"][j][i] * alphas[i]
        alphas.append(x - _map(x, _sum(xy, m, x), ks, gm))
    y = x0.clone()
    for a in alphas:
        y -= a
    return y
