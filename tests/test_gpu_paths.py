"""Kernel forms that the library chooses between by size: each at the sizes
where its tiles end, against the direct sum or against another form."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lf():
    import paper_2211_00354_amd as lf
    torch.cuda.set_device(0)
    return lf


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("p", [4, 8, 12, 15, 17, 24, 30, 36])
def test_m2l_forms_agree_bit_for_bit(lf, p, precision):
    # 256^2 leaf boxes of rays (1024 tiles: the form for many tiles) against
    # bands of 18 rows of boxes (96 tiles: the form for few), ragged at their
    # ends.  Every form adds each output's MFMA products in the same order, so
    # the outputs are equal bits; p covers every K-step count.
    f = wl.random_field(3000, 30.0, seed=41, masses="powerlaw")
    g = lf.Grid(-32.0, -32.0, 0.125, 0.125, 512, 512)
    xy, m = dev(f.xy), dev(f.m)
    plan = lf.Plan(xy, m, grid=g, precision=precision, p=p, leaf_level=8)
    whole = lf.deflect(plan=plan, grid=g)
    for j0 in range(0, 512, 35):
        ny = min(35, 512 - j0)
        band = lf.Grid(g.x0, g.y0 + j0 * g.dy, g.dx, g.dy, g.nx, ny)
        part = lf.deflect(plan=plan, grid=band)
        assert torch.equal(part, whole[j0 * 512:(j0 + ny) * 512]), (p, precision, j0)
    plan.close()
    if precision == "fp64" and p >= 30:
        ref = lf.deflect(xy, m, grid=g, method="direct")
        # truncation: the interaction list's ratio is at most 0.55, 0.55^30 = 2e-8
        # of a box's field; sums cancel below that
        assert float((whole - ref).norm() / ref.norm()) < 1e-8


@pytest.mark.parametrize("p", [24, 26, 36, 40])
@pytest.mark.parametrize("n,leaf", [(40, 2), (3000, 3), (3000, 5), (20000, 4), (20000, 7), (300000, 6)])
def test_p2m_lanes_and_shift_chains(lf, n, leaf, p):
    # 16 to 16384 leaf boxes of a fraction of a source to ~75 each (P2M with
    # 1, 4, 16 and 64 lanes per box), 1 to 6 levels of M2M and L2L above them,
    # and one leaf box of 3000 more sources with no level below it.  Truncation:
    # a source of the interaction list is at least 2 sides from the target's
    # centre, the target at most 0.71, the multipole's sources within 0.71 of
    # theirs, so terms fall by (1.41 / 2)^p at worst and by ~0.55^p on the mean
    # over a box; the field's own scale divides out.
    f = wl.random_field(n, 30.0, seed=43 + leaf, masses="powerlaw", kappa_s=0.1, gamma=0.2)
    rng = np.random.default_rng(5)
    xy = np.concatenate([f.xy, np.array([7.3, -4.1]) + 0.02 * rng.standard_normal((3000, 2))])
    m = np.concatenate([f.m, np.full(3000, 0.01)])
    g = lf.Grid(-32.0, -32.0, 1.0, 1.0, 64, 64)
    kw = dict(grid=g, kappa_s=f.kappa_s, gamma=f.gamma)
    ref = lf.deflect(dev(xy), dev(m), method="direct", **kw)
    y = lf.deflect(dev(xy), dev(m), precision="fp64", p=p, leaf_level=leaf, **kw)
    assert float((y - ref).norm() / ref.norm()) < 4 * 0.55 ** p


@pytest.mark.parametrize("precision,p,tol", [("fp64", 36, 1e-8), ("mixed", 24, 1e-4)])
@pytest.mark.parametrize("max_iter", [0, 1, 7, 8, 9, 40, 80])
def test_newton_iterations_match_direct(lf, max_iter, precision, p, tol):
    # the iterations run 8, then up to 64 to a launch; the direct sum steps one
    # at a time.  Both stop at the first iteration that leaves no candidate
    # above tol, or after max_iter, so they keep the same images; positions
    # within the evaluations' difference over |det A| (at most 1e3 here).
    f = wl.random_field(300, 30.0, seed=51, gamma=0.15)
    g = lf.Grid(-24.0, -24.0, 0.1875, 0.1875, 256, 256)
    xy, m = dev(f.xy), dev(f.m)
    src = dev(np.random.default_rng(3).uniform(-5, 5, (4, 2)))
    kw = dict(grid=g, sources=src, gamma=0.15, tol=tol, max_iter=max_iter)
    ref, rs = lf.find_images(xy, m, method="direct", **kw)
    img, s = lf.find_images(xy, m, precision=precision, p=p, **kw)
    ref, rs, img, s = (t.cpu().numpy() for t in (ref, rs, img, s))
    ok = np.abs(ref[:, 2]) < 1e3
    assert abs(len(img) - len(ref)) <= (0 if precision == "fp64" else 1 + len(ref) // 50)
    for r, k in zip(ref[ok], rs[ok]):
        d = np.hypot(img[s == k, 0] - r[0], img[s == k, 1] - r[1])
        assert d.min(initial=np.inf) < 1e3 * (1e-9 if precision == "fp64" else tol)


@pytest.mark.parametrize("npix", [1, 2, 3, 5, 8, 101, 258])
def test_ipm_map_edges_of_tiles(lf, npix):
    # the row differences of wide cells lie in 4 x 2 tiles and k_ipm's sums in
    # segments of 8 pixels: maps that end inside them.  Same corners as the
    # oracle's; contributions round to 2^-40 of a pixel's magnification, a
    # pixel takes at most a few thousand of them.
    import oracle
    f, g, _ = wl.small_disk()
    side = 0.02 * npix if npix > 8 else 0.4  # cells of 1 to ~1000 pixels' images
    md = lf.MapDesc(-0.5 * side, -0.4 * side, side, npix)
    grid = lf.Grid(g.x0, g.y0, g.dx, g.dy, g.nx, g.ny)
    kw = dict(grid=grid, kappa_s=f.kappa_s, gamma=f.gamma, method="direct")
    xy, m = dev(f.xy), dev(f.m)
    mu = lf.ipm_map(xy, m, map=md, **kw).cpu().numpy()
    y = lf.deflect(xy, m, **kw).cpu().numpy()
    ref = oracle.ipm(y.reshape(g.ny, g.nx, 2), g.dx * g.dy, md.y1min, md.y2min, md.side, npix)
    assert np.abs(mu - ref).max() <= 1e-9 * max(1.0, ref.max())
    again = lf.ipm_map(xy, m, map=md, max_rays_per_chunk=41 * g.nx, **kw).cpu().numpy()
    np.testing.assert_array_equal(mu, again)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 17, 1001])
@pytest.mark.parametrize("nx,ny", [(1, 1), (63, 1), (65, 3), (725, 724), (1024, 513)])
def test_direct_sum_forms(lf, n, nx, ny):
    # the stars shared out over a workgroup's waves (up to 524288 rays) and
    # whole (725 * 724 = 524900, 1024 * 513), counts that leave slices empty;
    # against the oracle on a sample.  Each pair carries a few FP64 roundings
    # of its own size, so the error is bounded by the sum of the pairs' sizes.
    import oracle
    f = wl.random_field(n, 10.0, seed=60 + n, masses="powerlaw", kappa_s=0.1, gamma=0.2)
    g = lf.Grid(-6.0, -6.0, 12.0 / nx, 12.0 / ny, nx, ny)
    y, d = lf.deflect(dev(f.xy), dev(f.m), grid=g, kappa_s=0.1, gamma=0.2, method="direct", want_dfdz=True)
    y1 = lf.deflect(dev(f.xy), dev(f.m), grid=g, kappa_s=0.1, gamma=0.2, method="direct")
    assert torch.equal(y, y1)
    w = wl.Grid(g.x0, g.y0, g.dx, g.dy, nx, ny)
    idx = np.unique(np.linspace(0, nx * ny - 1, 64).astype(np.int64))
    rays = w.rays(idx)
    yo, _, _ = oracle.deflect(f.xy, f.m, rays, 0.1, 0.2)
    z = rays[:, :1] + 1j * rays[:, 1:] - (f.xy[:, 0] + 1j * f.xy[:, 1])[None, :]
    size = (f.m / np.abs(z)).sum(1) + 12.0
    got = y.cpu().numpy()[idx]
    assert (np.abs(got - yo).max(1) <= 16 * np.finfo(float).eps * size).all()
    fp = -(f.m / z ** 2).sum(1)
    size2 = (f.m / np.abs(z) ** 2).sum(1)
    dz = d.cpu().numpy()[idx]
    assert (np.abs(dz[:, 0] + 1j * dz[:, 1] - fp) <= 32 * np.finfo(float).eps * size2).all()


@pytest.mark.parametrize("n", [1, 2, 64, 65, 1023, 1025, 8192, 8193, 20000, 524287, 524288, 2200000])
@pytest.mark.parametrize("leaf", [2, 7, 8])
def test_tree_sort_forms(lf, n, leaf):
    # one workgroup (up to 8192 points in 16384 boxes), radix passes over 2048-
    # and 4096-point tiles, packed records from 2^19 points: the sorted stars
    # give each box its multipole, so rays far outside every box's near field
    # see the field of all of them, and a plan's backward pass returns gradients
    # in the caller's order.
    rng = np.random.default_rng(n + leaf)
    xy = rng.uniform(-8, 8, (n, 2))
    m = rng.uniform(0.5, 1.5, n)
    xy[: min(n, 3)] = xy[0]  # equal keys
    rays = dev(np.array([[9.0, 0.25], [-0.75, 10.0], [0.3, 0.2], [-7.9, 7.7]]))
    box = (-10.0, -10.0, 10.0, 10.0)
    X, M = dev(xy), dev(m)
    plan = lf.Plan(X, M, ray_box=box, precision="fp64", p=40, leaf_level=leaf)
    y = lf.deflect(rays=rays, plan=plan)
    ref = lf.deflect(X, M, rays=rays, method="direct")
    assert float((y - ref).norm() / (ref - rays).norm()) < 1e-9
    g = dev(rng.standard_normal((4, 2)))
    gx, gm = lf.deflect_backward(None, None, g, rays=rays, plan=plan)
    rx, rm = lf.deflect_backward(X, M, g, rays=rays, method="direct")
    plan.close()
    assert float((gx - rx).norm() / rx.norm()) < 1e-8
    assert float((gm - rm).norm() / rm.norm()) < 1e-8


@pytest.mark.parametrize("precision,tol", [("mixed", 1e-5), ("fp64", 1e-9)])
@pytest.mark.parametrize("n,n_rays,radius", [
    (1, 1, 1.0), (63, 400, 30.0), (300, 70000, 30.0), (16385, 20000, 30.0), (20000, 40000, 2.0),
    (65537, 30000, 30.0), (65537, 60000, 3.0), (70000, 90000, 2.0)])
def test_adjoint_lanes_per_target(lf, n, n_rays, radius, precision, tol):
    # one, four and sixteen lanes to a star, by the number of stars and by how
    # many rays share a box; every neighbourhood size around the groups of
    # sources occurs between a dense middle and an empty rim.  Two stars lie on
    # rays (such pairs add nothing).
    f = wl.random_field(n, 30.0, seed=n, masses="powerlaw")
    rng = np.random.default_rng(n_rays)
    rays = (rng.random((n_rays, 2)) - 0.5) * 2 * radius
    xy = f.xy.copy()
    k = min(2, n, n_rays)
    xy[:k] = rays[:k]
    X, M, r = dev(xy), dev(f.m), dev(rays)
    g = dev(rng.standard_normal((n_rays, 2)))
    rx, rm = lf.deflect_backward(X, M, g, rays=r, method="direct")
    p = 12 if precision == "mixed" else 24
    plan = lf.Plan(X, M, ray_box=(-31.0, -31.0, 31.0, 31.0), precision=precision, p=p)
    for gx, gm in (lf.deflect_backward(X, M, g, rays=r, precision=precision, p=p),
                   lf.deflect_backward(None, None, g, rays=r, plan=plan)):
        for a, b in ((gx, rx), (gm, rm)):
            # a box without rays near it has locals of every ray at one size:
            # the norm over all stars is the scale
            assert float((a - b).norm()) <= tol * max(float(b.norm()), 1e-300)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("n,leaf_level,side", [(5, 3, 16), (3000, 3, 96), (3000, 5, 33), (20000, 4, 130)])
def test_explicit_rays_match_grid(lf, n, leaf_level, side, precision):
    # a lane to a ray against a wave to a box: the same rays as a grid and as
    # points, shuffled.  A core of stars gives some neighbourhoods thousands of
    # them (many moves of the FP32 sums), others a few or none.  Both add the
    # same pairs in the same order; the FP64 sums behind them may round a few
    # times otherwise (1e-14 of the largest value).
    f = wl.random_field(n, 30.0, seed=n + side, masses="powerlaw")
    xy = f.xy.copy()
    xy[: n // 2] *= 0.1
    X, M = dev(xy), dev(f.m)
    g = lf.Grid(-31.0, -30.5, 61.0 / side, 60.0 / side, side, side)
    plan = lf.Plan(X, M, ray_box=(-32.0, -32.0, 32.0, 32.0), precision=precision, p=12, leaf_level=leaf_level)
    i, j = np.meshgrid(np.arange(side), np.arange(side))
    r = np.stack([g.x0 + (i + 0.5) * g.dx, g.y0 + (j + 0.5) * g.dy], -1).reshape(-1, 2)
    order = np.random.default_rng(side).permutation(len(r))
    rays = dev(r[order])
    d, dg = (torch.empty((len(r), 2), dtype=torch.float64, device="cuda") for _ in range(2))
    yg, _ = lf.deflect(plan=plan, grid=g, dfdz_out=dg)
    for deriv in (False, True):
        y = lf.deflect(plan=plan, rays=rays, dfdz_out=d)[0] if deriv else lf.deflect(plan=plan, rays=rays)
        ref = yg.reshape(-1, 2)[dev(order)]
        assert float((y.reshape(-1, 2) - ref).abs().max()) <= 1e-14 * float(ref.abs().max())
    ref = dg[dev(order)]
    assert float((d - ref).abs().max()) <= 1e-14 * float(ref.abs().max())


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_bounds_of_rays(lf, bad):
    # the box of LensDeflect's rays: exact, and refused as soon as one
    # coordinate of many is not finite
    import ctypes

    from paper_2211_00354_amd import _lib
    for n in (1, 255, 70001):
        r = torch.randn((n, 2), dtype=torch.float64, device="cuda")
        out = (ctypes.c_double * 4)()
        _lib.check(_lib.load().lens_bounds(r.data_ptr(), n, out, None))
        assert tuple(out) == (*r.amin(0).tolist(), *r.amax(0).tolist())
        r[n // 2, 1] = bad
        one = torch.ones((1, 2), dtype=torch.float64, device="cuda")
        with pytest.raises(RuntimeError):
            lf.LensDeflect.apply(one, one[:, 0].contiguous(), r)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 7, 12, 17, 24, 31, 40])
@pytest.mark.parametrize("nx,ny,leaf_level", [(64, 64, 2), (65, 63, 2), (126, 251, 3), (521, 333, 4), (37, 1, 2)])
def test_mirrored_rays_match_points(lf, nx, ny, leaf_level, p, precision):
    # grids whose boxes hold enough rays for four mirror images to a lane (and,
    # last, one that is a single row): even and odd boxes, aligned ones and
    # others, boxes cut off at the grid's end; against the same rays as points.
    # The pairs are added in the same order; the far fields are two FP64 sums
    # of at most 40 decreasing terms, the shared one with a recurrence that
    # damps its roundings eightfold at worst, so 1e-13 of the largest value
    # covers 40 roundings of either twice.
    f = wl.random_field(2000, 30.0, seed=nx + p, masses="powerlaw")
    X, M = dev(f.xy), dev(f.m)
    g = lf.Grid(-31.0, -30.5, 61.0 / nx, 60.0 / ny, nx, ny)
    plan = lf.Plan(X, M, grid=g, precision=precision, p=p, leaf_level=leaf_level)
    i, j = np.meshgrid(np.arange(nx), np.arange(ny))
    r = np.stack([g.x0 + (i + 0.5) * g.dx, g.y0 + (j + 0.5) * g.dy], -1).reshape(-1, 2)
    yg = lf.deflect(plan=plan, grid=g).reshape(-1, 2)
    y = lf.deflect(plan=plan, rays=dev(r)).reshape(-1, 2)
    assert float((y - yg).abs().max()) <= 1e-13 * float(y.abs().max())
    # f' too (its terms grow by up to p against f's); y is the same bits with it
    y2, dg = lf.deflect(plan=plan, grid=g, want_dfdz=True)
    _, d = lf.deflect(plan=plan, rays=dev(r), want_dfdz=True)
    assert torch.equal(y2.reshape(-1, 2), yg)
    scale = max(float(d.abs().max()), float(y.abs().max()))
    assert float((d.reshape(-1, 2) - dg.reshape(-1, 2)).abs().max()) <= 1e-13 * p * scale
    # the same sums binned into a map
    npix = 64
    counts = lf.irs_map(plan=plan, grid=g, map=lf.MapDesc(-20.0, -20.0, 40.0, npix))
    t = torch.floor((yg + 20.0) * (npix / 40.0)).long()
    ok = ((t >= 0) & (t < npix)).all(1)
    ref = torch.bincount(t[ok, 1] * npix + t[ok, 0], minlength=npix * npix).reshape(npix, npix)
    assert int((counts.reshape(npix, npix) - ref).abs().sum()) <= 2


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_mirrored_rays_in_bands(lf, precision):
    # a call cut into bands of rows (a caller's buffer that holds part of the
    # locals) that end inside boxes of mirrored rays: the bits of the whole call
    from paper_2211_00354_amd import _lib
    f = wl.random_field(2000, 30.0, seed=3, masses="powerlaw")
    g = lf.Grid(-31.0, -30.5, 61.0 / 521, 60.0 / 333, 521, 333)
    plan = lf.Plan(dev(f.xy), dev(f.m), grid=g, precision=precision, p=12, leaf_level=4)
    y, d = lf.deflect(plan=plan, grid=g, want_dfdz=True)
    ran = 0
    for kib in range(8, 96, 4):
        ws = torch.empty(kib << 10, dtype=torch.uint8, device="cuda")
        try:
            yb, db = lf.deflect(plan=plan, grid=g, want_dfdz=True, workspace=ws)
        except _lib.LensError as e:
            assert e.status == _lib.LENS_ENOMEM
            continue
        ran += 1
        assert torch.equal(y, yb) and torch.equal(d, db)
        assert torch.equal(lf.deflect(plan=plan, grid=g, workspace=ws), y)
    assert ran >= 4


@pytest.mark.parametrize("n", [3, 31, 32, 35, 1000])
def test_direct_sum_does_not_depend_on_the_passes(lf, n):
    # 716800 rays at once (a wave's rays to itself) and in passes on the other
    # side of 524288 (the stars shared over four waves): equal bits
    f = wl.random_field(n, 10.0, seed=70 + n, masses="powerlaw", kappa_s=0.1, gamma=0.2)
    X, M = dev(f.xy), dev(f.m)
    g = lf.Grid(-6.0, -6.0, 12.0 / 1024, 12.0 / 700, 1024, 700)
    kw = dict(kappa_s=0.1, gamma=0.2, method="direct")
    y = lf.deflect(X, M, grid=g, **kw)
    i, j = np.meshgrid(np.arange(g.nx), np.arange(g.ny))
    rays = dev(np.stack([g.x0 + (i + 0.5) * g.dx, g.y0 + (j + 0.5) * g.dy], -1).reshape(-1, 2))
    parts = [lf.deflect(X, M, rays=rays[k:k + 300000], **kw) for k in range(0, len(rays), 300000)]
    assert torch.equal(torch.cat(parts), y)
    npix = 257
    ipm = dict(grid=g, map=lf.MapDesc(-4.0, -4.0, 8.0, npix), **kw)
    assert torch.equal(lf.ipm_map(X, M, **ipm), lf.ipm_map(X, M, max_rays_per_chunk=200 * 1024, **ipm))
    assert torch.equal(lf.irs_map(X, M, **ipm), lf.irs_map(X, M, max_rays_per_chunk=200 * 1024, **ipm))


def test_direct_sum_of_almost_2_32_rays(lf):
    # a launch takes fewer than 2^32 threads: 2^32 - 4 rays (the most a call
    # takes are 2^32 - 2) without stars, 64 GiB of y, are more than one
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 64 GiB of device memory")
    nx, ny = (1 << 30) - 1, 4
    n = nx * ny
    g = lf.Grid(-1.0, -2.0, 2.0 / nx, 1.0, nx, ny)
    none = torch.empty((0, 2), dtype=torch.float64, device="cuda")
    y = torch.full((n, 2), float("nan"), dtype=torch.float64, device="cuda")
    lf.deflect(none, none[:, 0].contiguous(), grid=g, gamma=0.25, out=y)
    for k in (0, nx, (1 << 31) - 1, 1 << 31, (1 << 31) + 256, n - 257, n - 1):
        i, j = k % nx, k // nx
        x = ((g.x0 + (i + 0.5) * g.dx) * 0.75, (g.y0 + (j + 0.5) * g.dy) * 1.25)
        assert tuple(y[k].tolist()) == x
    assert not bool(torch.isnan(y[:: 1 << 12, 0]).any())
    del y
    torch.cuda.empty_cache()


def test_adjoint_of_2_28_stars(lf):
    # sixteen lanes to a star would be 2^32 threads, which no launch takes: 2^28
    # stars on 8192 rays in 16 boxes, against the backward pass of a few of them
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs about 40 GiB of device memory")
    n = 1 << 28
    gen = torch.Generator(device="cuda").manual_seed(5)
    xy = torch.rand((n, 2), generator=gen, dtype=torch.float64, device="cuda").mul_(64.0).sub_(32.0)
    m = torch.ones(n, dtype=torch.float64, device="cuda")
    rays = torch.rand((8192, 2), generator=gen, dtype=torch.float64, device="cuda").mul_(64.0).sub_(32.0)
    g = torch.randn((8192, 2), generator=gen, dtype=torch.float64, device="cuda")
    kw = dict(rays=rays, precision="fp64", p=24, leaf_level=2)
    gx, gm = lf.deflect_backward(xy, m, g, **kw)
    k = torch.arange(0, n, 65537, device="cuda")
    few = (xy[k].contiguous(), m[k].contiguous())
    rx, rm = lf.deflect_backward(*few, g, method="direct", rays=rays)
    # each star against the size of its own sums; truncation 4 * 0.55^24 of them
    d2 = torch.cdist(few[0], rays) ** 2
    size = g.norm(dim=1)
    tol = 4 * 0.55 ** 24
    assert bool(((gm[k] - rm).abs() <= tol * (size / d2.sqrt()).sum(1)).all())
    assert bool(((gx[k] - rx).norm(dim=1) <= 24 * tol * (size / d2).sum(1)).all())
    del xy, m, gx, gm
    torch.cuda.empty_cache()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("n,leaf_level", [(1, 2), (2048, 2), (2049, 2), (3000, 7), (20000, 3), (20000, 6)])
def test_explicit_rays_do_not_depend_on_their_number(lf, n, leaf_level, precision):
    # one, four and sixteen lanes to a ray (70000, 65536 and 8192 rays), whose
    # neighbourhoods hold no star to thousands: groups of stars that end before,
    # at and after the end of a row, the last one empty or not.  Equal bits.
    f = wl.random_field(n, 30.0, seed=n + leaf_level, masses="powerlaw")
    xy = f.xy.copy()
    xy[: n // 2] *= 0.1
    X, M = dev(xy), dev(f.m)
    plan = lf.Plan(X, M, ray_box=(-32.0, -32.0, 32.0, 32.0), precision=precision, p=12, leaf_level=leaf_level)
    rays = dev(np.random.default_rng(n).uniform(-31, 31, (70000, 2)))
    ref = lf.deflect(plan=plan, rays=rays, want_dfdz=True)
    for part in (65536, 8192, 5000):
        for deriv in (False, True):
            r = rays[:part].contiguous()
            got = lf.deflect(plan=plan, rays=r, want_dfdz=True) if deriv else (lf.deflect(plan=plan, rays=r),)
            for a, b in zip(got, ref):
                assert torch.equal(a, b[:part])
    # and the direct sum's values: pairs of 2^-24 (2^-53) of their size each, the
    # truncation 0.55^12 of the far field's
    direct = lf.deflect(X, M, rays=rays[:5000].contiguous(), method="direct")
    assert float((ref[0][:5000] - direct).norm() / direct.norm()) < 4 * 0.55 ** 12


@pytest.mark.parametrize("precision,p,tol,n_src", [("fp64", 30, 1e-9, 24), ("mixed", 16, 1e-4, 12)])
def test_images_of_many_candidates(lf, precision, p, tol, n_src):
    # ~900 candidates a source: all of them are more than a wave each takes, four
    # sources' are not.  The same images (but for those that converge only just),
    # each as far from the other form's as the residuals allow: 2 tol |mu|.
    f = wl.random_field(1000, 30.0, seed=52, gamma=0.1)
    g = lf.Grid(-32.0, -32.0, 0.125, 0.125, 512, 512)
    plan = lf.Plan(dev(f.xy), dev(f.m), grid=g, precision=precision, p=p)
    src = dev(np.random.default_rng(4).uniform(-3, 3, (n_src, 2)))
    kw = dict(plan=plan, grid=g, gamma=0.1, precision=precision, p=p, tol=tol)
    img, s = (t.cpu().numpy() for t in lf.find_images(sources=src, **kw))
    assert len(img) > (16384 if precision == "fp64" else 8192)
    odd = 0
    for k in range(0, n_src, 4):
        ref, rs = (t.cpu().numpy() for t in lf.find_images(sources=src[k:k + 4].contiguous(), **kw))
        for j in range(4):
            a, b = img[s == k + j], ref[rs == j]
            d = np.hypot(a[:, None, 0] - b[None, :, 0], a[:, None, 1] - b[None, :, 1])
            ok = np.abs(b[:, 2]) < 1e3
            near = d.min(0) <= 2 * tol * np.maximum(1.0, np.abs(b[:, 2])) * 4
            odd += int((~near & ok).sum()) + abs(len(a) - len(b))
    assert odd <= len(img) // 1000


@pytest.mark.parametrize("rows", [1, 2, 5, 40])
def test_ipm_short_queues(lf, rows):
    # wide cells (up to hundreds of pixels) in passes of a few rows of cells, whose
    # queues of tens to thousands of cells are shared out over 16 waves to one;
    # sums of integers, so the whole call's bits, and the oracle's values
    import oracle
    f, g, _ = wl.small_disk()
    grid = lf.Grid(g.x0, g.y0, g.dx, g.dy, g.nx, g.ny)
    npix = 700
    md = lf.MapDesc(-1.5, -1.4, 3.0, npix)
    kw = dict(grid=grid, map=md, kappa_s=f.kappa_s, gamma=f.gamma, method="direct")
    xy, m = dev(f.xy), dev(f.m)
    mu = lf.ipm_map(xy, m, **kw)
    assert torch.equal(mu, lf.ipm_map(xy, m, max_rays_per_chunk=(rows + 1) * g.nx, **kw))
    if rows == 1:
        y = lf.deflect(xy, m, grid=grid, kappa_s=f.kappa_s, gamma=f.gamma, method="direct").cpu().numpy()
        ref = oracle.ipm(y.reshape(g.ny, g.nx, 2), g.dx * g.dy, md.y1min, md.y2min, md.side, npix)
        assert np.abs(mu.cpu().numpy() - ref).max() <= 1e-9 * max(1.0, ref.max())


@pytest.mark.parametrize("p", [24, 40])
@pytest.mark.parametrize("off", [0.0, 3.0e5, 1.0e8])
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("nx,ny,leaf_level", [(256, 256, 3), (250, 250, 3), (1001, 777, 4)])
def test_mirrored_rays_far_from_the_origin(lf, nx, ny, leaf_level, aligned, off, p):
    # FP64: rays in boxes that the mirrored form fits, with exact coordinates
    # (256^2) and rounded ones, on boxes aligned with them and on others, against
    # the same rays as points.  y = -alpha; the pairs agree in all but the order of
    # their sums and the far fields are two sums of at most 40 terms at the same
    # place, so the bound of the rays near the origin holds wherever they are.
    f = wl.random_field(2000, 30.0, seed=nx + p, masses="powerlaw")
    xy = f.xy + off
    g = lf.Grid(off - 31.0, off - 30.5, 61.0 / nx, 60.0 / ny, nx, ny)
    where = {"grid": g} if aligned else {"ray_box": (off - 31.7, off - 31.3, off + 31.1, off + 30.9)}
    plan = lf.Plan(dev(xy), dev(f.m), precision="fp64", p=p, leaf_level=leaf_level, **where)
    i, j = np.meshgrid(np.arange(nx), np.arange(ny))
    r = dev(np.stack([g.x0 + (i + 0.5) * g.dx, g.y0 + (j + 0.5) * g.dy], -1).reshape(-1, 2))
    yg, dg = lf.deflect(plan=plan, grid=g, kappa_s=1.0, want_dfdz=True)
    y, d = lf.deflect(plan=plan, rays=r, kappa_s=1.0, want_dfdz=True)
    assert float((y - yg).abs().max()) <= 1e-13 * float(y.abs().max())
    scale = max(float(d.abs().max()), float(y.abs().max()))
    assert float((d - dg).abs().max()) <= 1e-13 * p * scale


def test_plans_keep_no_sort_records(lf):
    # of the packed records of a sort (32 bytes a star from 2^19 stars on) a plan
    # keeps none: the second of two plans takes its stars (28 bytes), the sort's
    # keys and values (16) and its boxes, and less where the pool has blocks
    n = 1 << 22
    xy = torch.rand((n, 2), dtype=torch.float64, device="cuda")
    m = torch.ones(n, dtype=torch.float64, device="cuda")
    plans = [lf.Plan(xy, m, ray_box=(0.0, 0.0, 1.0, 1.0), p=2, leaf_level=7)]
    torch.cuda.synchronize()
    for _ in range(3):
        free = torch.cuda.mem_get_info()[0]
        plans.append(lf.Plan(xy, m, ray_box=(0.0, 0.0, 1.0, 1.0), p=2, leaf_level=7))
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] <= 48 * n
    # the sorts shared the records; each has its own stars
    g = lf.Grid(0.25, 0.25, 0.01, 0.01, 8, 8)
    y = [lf.deflect(plan=p, grid=g) for p in plans]
    assert all(torch.equal(y[0], other) for other in y[1:])
    for p in plans:
        p.close()


@pytest.mark.parametrize("precision,p,eps", [("mixed", 20, 2.0 ** -24), ("fp64", 28, 2.0 ** -53)])
@pytest.mark.parametrize("n,n_rays,radius", [
    (300, 30000, 30.0), (16385, 20000, 30.0), (40000, 30000, 4.0), (65537, 20000, 3.0), (140000, 30000, 30.0)])
def test_adjoint_star_by_star(lf, n, n_rays, radius, precision, p, eps):
    # one, four and sixteen lanes to a star, each star against the size of its own
    # sums, sum |g| / |d| and m sum |g| / |d|^2 (a norm over all stars is that of a
    # few close pairs).  A pair carries a few roundings of its size; the far field
    # is truncated at 0.55^p of it, its derivative's terms grow by p.
    f = wl.random_field(n, 30.0, seed=n + 1, masses="powerlaw")
    rng = np.random.default_rng(n_rays + n)
    rays = (rng.random((n_rays, 2)) - 0.5) * 2 * radius
    X, M, r = dev(f.xy), dev(f.m), dev(rays)
    g = dev(rng.standard_normal((n_rays, 2)))
    rx, rm = lf.deflect_backward(X, M, g, rays=r, method="direct")
    plan = lf.Plan(X, M, ray_box=(-31.0, -31.0, 31.0, 31.0), precision=precision, p=p)
    got = (lf.deflect_backward(X, M, g, rays=r, precision=precision, p=p),
           lf.deflect_backward(None, None, g, rays=r, plan=plan))
    tol = 4 * 0.55 ** p + 64 * eps
    size = g.norm(dim=1)
    for a in range(0, n, 2000):
        k = slice(a, min(n, a + 2000))
        d = r[None] - X[k, None]
        d2 = (d * d).sum(-1)
        s1, s2 = (size / d2.sqrt()).sum(1), M[k] * (size / d2).sum(1)
        for gx, gm in got:
            assert bool(((gm[k] - rm[k]).abs() <= tol * s1).all())
            assert bool(((gx[k] - rx[k]).norm(dim=1) <= p * tol * s2).all())
        # the bound tells zero and a wrong sign from the gradient
        assert float((rx[k].norm(dim=1) > 2 * p * tol * s2).double().mean()) > 0.9
