"""Measured cases of the library: what a program has it do, over the sizes, fields and options in use.

A case is a dict of plain values.  ``kind`` names the call or the chain of calls:

* ``step``    isobands, components, Lloyd loop and three-level statistics of one volume (the library's main use);
* ``labels``  isobands, components and stratified initial sites: what a program runs once per new field;
* ``lloyd``   the Lloyd loop alone, on labels that the program has already;
* ``pass``    one Voronoi pass and one site update, for programs that drive their own loop;
* ``stats``   statistics of a finished tessellation;
* ``moments`` joint moments up to fourth order of a finished tessellation;
* ``layout``  structured layout and raw-data extraction;
* ``los``     the Lloyd loop with Euclidean line-of-sight paths;
* ``batch``   many uneven volumes in one call.

Fields are made on the GPU: ``blobs`` (Gaussians plus noise), ``fourier`` (random modes with a k^-5/3 spectrum) and
``flame`` (a thin wrinkled sheet with temperature and species), the three shapes that the package's generators and its
benchmark use.  The seed mirrors the volume along its axes (other labels, sites and cells, in tables of the same
lengths) and draws the noise of the variables.  Sites come from the library's own stratified seeding.
"""
import math

import numpy as np
import torch

import paper_2208_06970_amd as L


# --------------------------------------------------------------------------
# the cases
def listed():
    return [
        # the smallest whole step in use: a 64^3 block, uniform weight, launches and read-backs dominate
        {"name": "step_blobs_64", "kind": "step", "field": "blobs", "nx": 64, "ny": 64, "nz": 64, "iters": 10,
         "iso": 4, "vars": 3, "bins": 16, "cov": False, "rho": 512},
        # the turbulence-like benchmark volume: narrow cells, 8 variables, histograms and covariance
        {"name": "step_fourier_256", "kind": "step", "field": "fourier", "nx": 256, "ny": 256, "nz": 256, "iters": 20,
         "iso": 8, "vars": 8, "bins": 32, "cov": True, "rho": 4096},
        # the main benchmark workload: the largest volume, wide cells, 18 variables
        {"name": "step_flame_1024x512x512", "kind": "step", "field": "flame", "nx": 1024, "ny": 512, "nz": 512,
         "iters": 30, "iso": 10, "vars": 18, "bins": 32, "cov": True, "rho": 4096},
        # a new field of odd edges: bands, components and its initial sites
        {"name": "labels_501x333x187", "kind": "labels", "field": "fourier", "nx": 501, "ny": 333, "nz": 187,
         "iso": 6, "rho": 4096},
        # the Lloyd loop of one served job (edges 64..512, odd, 64 modes)
        {"name": "lloyd_379x251x147", "kind": "lloyd", "field": "fourier", "nx": 379, "ny": 251, "nz": 147,
         "iters": 20, "iso": 7, "rho": 4096},
        # one pass and one update of a 2:1:1 box of the batch's sizes
        {"name": "pass_192x96x96", "kind": "pass", "field": "fourier", "nx": 192, "ny": 96, "nz": 96, "iso": 5,
         "rho": 4096},
        # statistics of a flame block: 18 variables, histograms and the full covariance
        {"name": "stats_cov18_512x256x256", "kind": "stats", "field": "flame", "nx": 512, "ny": 256, "nz": 256,
         "iso": 10, "vars": 18, "bins": 32, "cov": True, "rho": 4096},
        # statistics of a small ragged block without covariance
        {"name": "stats_hist4_131x121x77", "kind": "stats", "field": "fourier", "nx": 131, "ny": 121, "nz": 77,
         "iso": 6, "vars": 4, "bins": 32, "cov": False, "rho": 4096},
        # coskewness and cokurtosis of the flame's 18 variables (7314 sums per voxel)
        {"name": "moments18_256x128x128", "kind": "moments", "field": "flame", "nx": 256, "ny": 128, "nz": 128,
         "iso": 10, "vars": 18, "rho": 4096},
        # reordering 8 raw variables by band, component and cell
        {"name": "layout8_333x255x201", "kind": "layout", "field": "fourier", "nx": 333, "ny": 255, "nz": 201,
         "iso": 8, "vars": 8, "rho": 4096},
        # the line-of-sight form of the tessellation
        {"name": "los_160x144x128", "kind": "los", "field": "fourier", "nx": 160, "ny": 144, "nz": 128, "iters": 3,
         "iso": 4, "rho": 512},
        # a quarter of the benchmark's batch: uneven volumes, edges 32..192
        {"name": "batch_16", "kind": "batch", "jobs": 16, "iters": 15, "vars": 8, "bins": 32, "cov": True,
         "rho": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _edges(rng, lo, hi, most):
    """Three edges, each log-uniform in [lo, hi], of a volume of at most `most` voxels."""
    while True:
        e = [_log_int(rng, lo, hi) for _ in range(3)]
        if e[0] * e[1] * e[2] <= most:
            return {"nx": e[0], "ny": e[1], "nz": e[2]}


def draw(rng):
    kind = rng.choice(["step", "step", "labels", "lloyd", "pass", "stats", "stats", "moments", "layout", "los",
                       "batch"])
    field = rng.choice(["fourier", "fourier", "flame", "blobs"])
    c = {"kind": kind, "field": field}
    rho = rng.choice([512, 1024, 4096])
    if kind == "step":
        c.update(_edges(rng, 48, 512, 1 << 25), iters=rng.randint(10, 30), iso=rng.randint(3, 12),
                 vars=rng.randint(3, 18), bins=rng.choice([16, 32]), cov=rng.random() < 0.7, rho=rho)
    elif kind == "labels":
        c.update(_edges(rng, 64, 512, 1 << 26), iso=rng.randint(3, 12), rho=rho)
    elif kind == "lloyd":
        c.update(_edges(rng, 64, 512, 1 << 25), iters=rng.randint(10, 30), iso=rng.randint(3, 12), rho=rho)
    elif kind == "pass":
        c.update(_edges(rng, 32, 256, 1 << 24), iso=rng.randint(3, 10), rho=rho)
    elif kind == "stats":
        c.update(_edges(rng, 64, 512, 1 << 25), iso=rng.randint(3, 12), vars=rng.randint(1, 18),
                 bins=rng.choice([0, 16, 32]), cov=rng.random() < 0.7, rho=rho)
    elif kind == "moments":
        m = rng.randint(1, 18)
        c.update(_edges(rng, 48, 256, 1 << 22), field="flame", iso=rng.randint(3, 10), vars=m, rho=4096)
    elif kind == "layout":
        c.update(_edges(rng, 64, 512, 1 << 25), iso=rng.randint(3, 12), vars=rng.randint(1, 16), rho=rho)
    elif kind == "los":
        c.update(_edges(rng, 32, 192, 3 << 20), iters=rng.randint(0, 4), iso=rng.randint(2, 6),
                 rho=rng.choice([256, 512, 1024]))
    else:
        c = {"kind": kind, "jobs": rng.randint(4, 24), "iters": rng.randint(5, 15), "vars": rng.randint(2, 8),
             "bins": 32, "cov": rng.random() < 0.7, "rho": rho}
    return c


# --------------------------------------------------------------------------
# inputs, on the GPU (elementwise operations in a fixed order: the same bits every time)
_GEOMETRY = 2  # the generator's seed: a case's table lengths do not depend on the seed it is prepared with


def _mirror(f, seed):
    """The volume reversed along the axes whose bits `seed` has set."""
    return f.flip([a for a in range(3) if seed >> a & 1]).contiguous()


def _wave(k, n):
    return torch.from_numpy(np.exp(2j * math.pi * np.outer(k, np.arange(n)) / n).astype(np.complex64)).cuda()


def _mode_sum(shape, seed, n_modes, kmax, box):
    """Random modes |k| in [1, kmax] cycles per `box` voxels, amplitude |k|^(-5/6), rescaled to [0, 1]."""
    rng = np.random.default_rng(seed)
    nz, ny, nx = shape
    kmag = rng.uniform(1.0, kmax, n_modes)
    d = rng.normal(size=(n_modes, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    c = kmag ** (-5.0 / 6.0) * np.exp(2j * math.pi * rng.uniform(size=n_modes))
    k = np.rint(kmag[:, None] * d * np.array([nx, ny, nz]) / box).astype(np.int64)
    kz = np.unique(k[:, 2])
    at = np.searchsorted(kz, k[:, 2])
    ex, ey, ez = _wave(k[:, 0], nx), _wave(k[:, 1], ny), _wave(kz, nz)
    ey *= torch.from_numpy(c.astype(np.complex64)).cuda()[:, None]
    plane = torch.zeros((len(kz), ny, nx), dtype=torch.complex64, device="cuda")
    for m in range(n_modes):
        plane[at[m]].addcmul_(ey[m][:, None], ex[m][None, :])
    re, im = plane.real.contiguous(), plane.imag.contiguous()
    del plane
    f = torch.zeros(shape, dtype=torch.float32, device="cuda")
    for j in range(len(kz)):
        f.addcmul_(ez[j].real[:, None, None], re[j][None])
        f.addcmul_(ez[j].imag[:, None, None], im[j][None], value=-1.0)
    lo, hi = f.min(), f.max()
    return f.sub_(lo).div_(torch.clamp(hi - lo, min=1e-30))


def _noise(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=g)


def _blobs(shape, seed):
    """Gaussians of 4 to 10 voxels (a few per 64^3 block, eight at least) plus 1 % noise."""
    rng = np.random.default_rng(seed)
    nz, ny, nx = shape
    f = _noise(shape, seed).mul_(0.01)
    for _ in range(min(64, max(8, nz * ny * nx >> 16))):
        s = 1.0 / (2.0 * rng.uniform(4.0, 10.0) ** 2)
        g = [torch.exp(-s * (torch.arange(n, device="cuda", dtype=torch.float32) - rng.uniform(0, n)) ** 2)
             for n in shape]
        f.addcmul_((g[0] * rng.uniform(0.5, 1.0))[:, None, None], (g[1][:, None] * g[2][None, :])[None])
    return f


def _gradient_weight(f):
    """max(1, round(65535 |grad f| / max |grad f|)) as 16 bits."""
    g = torch.zeros_like(f)
    for a in range(3):
        n = f.shape[a]
        if n >= 3:
            g.narrow(a, 1, n - 2).addcmul_(*[(f.narrow(a, 2, n - 2) - f.narrow(a, 0, n - 2)) * 0.5] * 2)
    g.sqrt_()
    g.mul_(65535.0 / torch.clamp(g.max(), min=1e-30)).round_().clamp_(1.0, 65535.0)
    return g.to(torch.int32).to(torch.int16)


def _isovalues(f, n):
    """Quantiles i / (n + 1) of an evenly spaced sample, strictly increasing."""
    v = f.reshape(-1)
    v = torch.sort(v[:: max(1, v.numel() >> 18)]).values.cpu().numpy()
    iso = v[[int(len(v) * (i + 1) / (n + 1)) for i in range(n)]].astype(np.float32)
    for i in range(1, n):
        if not iso[i - 1] < iso[i]:
            iso[i] = np.nextafter(iso[i - 1], np.float32(np.inf))
    return iso


def _flame(shape, seed, n_vars):
    """(Z, T, species ...) of a thin wrinkled sheet across y; at least the first two."""
    nz, ny, nx = shape
    s = _mode_sum(shape, _GEOMETRY, 512, 64.0, 512.0)
    s.mul_(0.1).sub_(0.05)
    s.add_((torch.arange(ny, device="cuda", dtype=torch.float32) / max(ny - 1, 1) - 0.5)[None, :, None])
    s = _mirror(s, seed)
    m = max(2, n_vars)
    x = torch.empty((m,) + tuple(shape), dtype=torch.float32, device="cuda")
    z = x[0]
    torch.tanh(s.div_(0.02), out=z)
    z.add_(1.0).mul_(0.5)
    torch.exp(((z - 0.3) / 0.1).square_().neg_(), out=x[1])
    x[1].mul_(1700.0).add_(300.0)
    if m > 2:
        g = _noise((z.numel(),), seed + 100).mul_(0.02)
        for i in range(m - 2):
            y = x[2 + i]
            torch.exp(((z - (i + 0.5) / 16) / (0.05, 0.1, 0.15, 0.2)[i % 4]).square_().neg_().clamp_(min=-80.0), out=y)
            y.view(-1).add_(torch.roll(g, 7919 * (i + 1)))
    return x


def _volume(c, seed):
    """Field, isovalues, weights (None: uniform) and variables of a case."""
    shape = (c["nz"], c["ny"], c["nx"])
    m = c.get("vars", 0)
    if c["field"] == "flame":
        x = _flame(shape, seed, m)
        f = x[0].clone()
        iso = np.array([(i + 0.5) / c["iso"] for i in range(c["iso"])], dtype=np.float32)
        return f, iso, _gradient_weight(x[1]), x[:m].contiguous() if m else None
    if c["field"] == "blobs":
        f = _blobs(shape, _GEOMETRY)
    else:
        modes = 512 if c["kind"] == "step" else 64
        f = _mode_sum(shape, c.get("geometry", _GEOMETRY), modes, 64.0, float(max(shape)))
    iso = _isovalues(f, c["iso"])
    f = _mirror(f, seed)
    x = None
    if m:
        # the field, then smooth functions of it with a little noise
        x = torch.empty((m,) + shape, dtype=torch.float32, device="cuda")
        x[0].copy_(f)
        for j in range(1, m):
            torch.sin(f * (2.0 + j) + 0.5 * j, out=x[j])
            x[j].mul_(1.0 + j).add_(_noise(shape, 1000 * (seed + 1) + j), alpha=0.05)
    return f, iso, None if c["field"] == "blobs" else _gradient_weight(f), x


def _histogram_edges(x, bins):
    if not bins:
        return None
    v = x.reshape(x.shape[0], -1)
    e = [np.linspace(float(a), float(b), bins + 1) for a, b in zip(v.min(1).values, v.max(1).values)]
    return torch.from_numpy(np.stack(e).astype(np.float32)).cuda()


def _sites(c, cc, w):
    return L.lsrvt_seed(cc.comp, cc.comp_first, cc.n_comp, w, rho=c["rho"], seed=0x5EED)


def _batch_specs(n, seed):
    """Long edge of {32, 48, ..., 192}, a cube or by coin a 2:1:1 box, 3..10 isovalues."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        e = int(rng.choice(np.arange(32, 193, 16)))
        s = [e, e, e]
        if rng.random() >= 0.5:
            s = [e // 2] * 3
            s[int(rng.integers(0, 3))] = e
        out.append((s, int(rng.integers(3, 11))))
    return out


def _tessellate(c, f, iso, w, iters):
    band, _ = L.lsrvt_isobands(f, iso)
    cc = L.lsrvt_components(band, len(iso) + 1)
    return band, cc, L.lsrvt_cvt(band, cc.comp, _sites(c, cc, w), w, iters)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c}
    if kind == "batch":
        s["jobs"] = []
        for j, ((nz, ny, nx), n_iso) in enumerate(_batch_specs(c["jobs"], 3)):  # the same sizes for every seed
            v = dict(c, kind="lloyd", field="fourier", nx=nx, ny=ny, nz=nz, iso=n_iso, geometry=3000 + j)
            f, iso, w, x = _volume(v, seed + j)
            cc = L.lsrvt_components(L.lsrvt_isobands(f, iso)[0], n_iso + 1)
            s["jobs"].append(dict(field=f, iso=iso, seeds=_sites(c, cc, w), weights=w, iters=c["iters"], variables=x,
                                  edges=_histogram_edges(x, c["bins"]), cov=c["cov"], cap_comp=cc.n_comp + 16))
        return s
    f, iso, w, x = _volume(c, seed)
    s.update(iso=iso, n_bands=len(iso) + 1, w=w)
    if kind == "labels":
        s["f"] = f
    elif kind == "step":
        cc = L.lsrvt_components(L.lsrvt_isobands(f, iso)[0], len(iso) + 1)
        s.update(f=f, x=x, edges=_histogram_edges(x, c["bins"]), seeds=_sites(c, cc, w))
    elif kind in ("lloyd", "pass", "los"):
        band, _ = L.lsrvt_isobands(f, iso)
        cc = L.lsrvt_components(band, len(iso) + 1)
        s.update(band=band, comp=cc.comp, seeds=_sites(c, cc, w))
    else:  # a finished tessellation
        band, cc, r = _tessellate(c, f, iso, w, 5)
        s.update(cell=r.cell, sites=r.sites, site_comp=r.site_comp, comp_band=cc.comp_band, n_comp=cc.n_comp, x=x,
                 edges=_histogram_edges(x, c.get("bins", 0)))
    return s


# --------------------------------------------------------------------------
# one pass
def _level(v):
    return {k: getattr(v, k) for k in ("n", "mean", "m2", "vmin", "vmax", "hist", "cov")}


def _stats(v):
    return {"cell": _level(v[0]), "comp": _level(v[1]), "band": _level(v[2])}


def _joint(v):
    return {k: getattr(v, k) for k in ("n", "mean", "m2", "m3", "m4")}


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "step":
        band, status = L.lsrvt_isobands(s["f"], s["iso"])
        cc = L.lsrvt_components(band, s["n_bands"])
        r = L.lsrvt_cvt(band, cc.comp, s["seeds"], s["w"], c["iters"])
        st = L.lsrvt_aggregate(r.cell, r.sites, r.site_comp, cc.comp_band, cc.n_comp, s["n_bands"], s["x"], s["edges"],
                               cov=c["cov"])
        return {"band": band, "status": status, "comp": cc.comp, "comp_band": cc.comp_band, "comp_size": cc.comp_size,
                "comp_first": cc.comp_first, "band_offset": cc.band_offset, "cells": r.cell, "sites": r.sites,
                "site_comp": r.site_comp, "mean_ds": r.mean_ds, **_stats(st)}
    if kind == "labels":
        band, status = L.lsrvt_isobands(s["f"], s["iso"])
        cc = L.lsrvt_components(band, s["n_bands"])
        return {"band": band, "status": status, "comp": cc.comp, "comp_band": cc.comp_band, "comp_size": cc.comp_size,
                "comp_first": cc.comp_first, "band_offset": cc.band_offset, "sites": _sites(c, cc, s["w"])}
    if kind == "lloyd":
        r = L.lsrvt_cvt(s["band"], s["comp"], s["seeds"], s["w"], c["iters"])
        return {"cells": r.cell, "sites": r.sites, "site_comp": r.site_comp, "mean_ds": r.mean_ds}
    if kind == "pass":
        cell = L.lsrvt_vt(s["band"], s["seeds"])
        sites, ds = L.lsrvt_update(cell, s["seeds"].clone(), s["w"])  # the update moves its sites in place
        return {"cells": cell, "sites": sites, "ds": ds}
    if kind == "stats":
        return _stats(L.lsrvt_aggregate(s["cell"], s["sites"], s["site_comp"], s["comp_band"], s["n_comp"],
                                        s["n_bands"], s["x"], s["edges"], cov=c["cov"]))
    if kind == "moments":
        cm, gm, bm = L.lsrvt_comoments(s["cell"], s["sites"], s["site_comp"], s["comp_band"], s["n_comp"],
                                       s["n_bands"], s["x"])
        return {"cell": _joint(cm), "comp": _joint(gm), "band": _joint(bm)}
    if kind == "layout":
        lay = L.lsrvt_layout(s["cell"], s["site_comp"], s["comp_band"], s["n_comp"], s["n_bands"])
        return {"perm": lay.perm, "site_order": lay.site_order, "cell_off": lay.cell_off, "comp_off": lay.comp_off,
                "band_off": lay.band_off, "raw": L.lsrvt_extract(s["x"], lay.perm)}
    if kind == "los":
        r = L.lsrvt_los_cvt(s["comp"], s["seeds"], s["w"], c["iters"])
        return {"site_q": r.site_q, "anchor": r.anchor, "dist": r.vt.dist, "src": r.vt.src, "phi": r.vt.phi,
                "cells": r.vt.cell, "sweeps": list(r.vt.sweeps)}
    jobs = L.lsrvt_batch_run([L.BatchJob(**j) for j in s["jobs"]])
    out = {}
    for k in ("band", "comp", "cell", "sites", "site_comp", "band_offset"):
        out[k] = torch.cat([getattr(j, k).reshape(-1) for j in jobs])
    for k in ("comp_band", "comp_size", "comp_first"):
        out[k] = torch.cat([getattr(j, k)[:j.n_comp] for j in jobs])
    for i, level in enumerate(("cells", "comps", "bands")):
        for k in ("n", "mean", "m2", "vmin", "vmax", "hist", "cov"):
            v = [getattr(j.stats[i], k) for j in jobs]
            if v[0] is not None:
                out[level + "_" + k] = torch.cat([(a[:j.n_comp] if i == 1 else a).reshape(-1)
                                                  for a, j in zip(v, jobs)])
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
def _voxels(c):
    if c["kind"] == "batch":
        return sum(nz * ny * nx for (nz, ny, nx), _ in _batch_specs(c["jobs"], 3))
    return c["nx"] * c["ny"] * c["nz"]


def work(case):
    """Inputs read once and outputs written once, per voxel (tables of sites and components are small beside them),
    and the multiply-adds of the moments' sums."""
    c, kind, n, m = case, case["kind"], _voxels(case), case.get("vars", 0)
    sums = m + (m * (m + 1) // 2 if c.get("cov") else m)
    w = 0 if c.get("field") == "blobs" else 2
    if kind in ("step", "batch"):
        return {"bytes": n * (4 + w + 4 * m + 1 + 4 + 4), "flops": 2 * n * sums}
    if kind == "labels":
        return {"bytes": n * (4 + w + 1 + 4), "flops": 0}
    if kind == "lloyd":
        return {"bytes": n * (1 + w + 4), "flops": 0}
    if kind == "pass":
        return {"bytes": n * (1 + w + 4), "flops": 0}
    if kind == "stats":
        return {"bytes": n * (4 + 4 * m), "flops": 2 * n * sums}
    if kind == "moments":
        units = math.comb(m + 4, 4) - 1
        return {"bytes": n * (4 + 4 * m), "flops": 2 * n * units}
    if kind == "layout":
        return {"bytes": n * (4 + 4 + 8 * m), "flops": 0}
    return {"bytes": n * (4 + w + 8 + 4 + 4 + 4), "flops": 0}


# --------------------------------------------------------------------------
# the floating outputs in 64 bits, by plain torch
def _units(cell, site_comp, comp_band):
    """Flat indices of the placed voxels ordered by component, cell and index (components are numbered by band), and
    the cell, component and band of each: every unit is one run of consecutive voxels."""
    at = torch.nonzero(cell.reshape(-1) != -1).reshape(-1)
    u = cell.reshape(-1)[at].long()
    g = site_comp.long()[u]
    order = torch.argsort(g * site_comp.numel() + u, stable=True)
    at, u, g = at[order], u[order], g[order]
    return at, (u, g, comp_band.long()[g])


def _blocks(unit, size=64):
    """Consecutive equal entries of `unit` cut into blocks of `size`: index matrix (-1: padding) and each block's
    unit."""
    ids, count = torch.unique_consecutive(unit, return_counts=True)
    per = (count + size - 1) // size
    start = torch.cumsum(count, 0) - count
    own = torch.repeat_interleave(torch.arange(ids.numel(), device="cuda"), per)
    k = torch.arange(own.numel(), device="cuda") - torch.repeat_interleave(torch.cumsum(per, 0) - per, per)
    at = start[own][:, None] + k[:, None] * size + torch.arange(size, device="cuda")
    return torch.where(at < (start + count)[own][:, None], at, -1), ids[own]


def _tuples(m, k):
    """Index tuples i <= j <= ... of length k over m variables, lexicographic."""
    t = [()]
    for _ in range(k):
        t = [a + (i,) for a in t for i in range(a[-1] if a else 0, m)]
    return torch.tensor(t, device="cuda").T


def _reduce(unit, n_units, columns, values, op, empty):
    """op over the rows of every unit, in blocks of 64 rows and then blocks of blocks.  values(i, u): the float64 rows
    [len(u), 64, columns] of the index matrix i, whose blocks belong to the units u."""
    while True:
        at, own = _blocks(unit)
        rows = torch.empty((own.numel(), columns), dtype=torch.float64, device="cuda")
        step = max(64, (1 << 21) // columns)
        for i in range(0, own.numel(), step):
            a = at[i:i + step]
            v = torch.where((a >= 0)[:, :, None], values(a.clamp(min=0), own[i:i + step]), empty)
            rows[i:i + step] = op(v)
        if torch.unique_consecutive(own).numel() == own.numel():
            break
        unit, values = own, lambda a, u, rows=rows: rows[a]
    out = torch.full((n_units, columns), empty, dtype=torch.float64, device="cuda")
    out[own] = rows
    return out


def _centred(at, unit, n_units, x, orders, extrema=False):
    """Means, centred sums of each order in `orders` and extrema of every unit, in float64."""
    m = x.shape[0]
    v = x.reshape(m, -1)
    total = lambda t: t.sum(1)
    plain = lambda a, u: v[:, at[a]].double().permute(1, 2, 0)
    mean = _reduce(unit, n_units, m, plain, total, 0.0)
    mean /= torch.bincount(unit, minlength=n_units).clamp(min=1)[:, None]
    out = {}
    for k in orders:
        t = _tuples(m, k)

        def product(a, u):
            d = plain(a, u) - mean[u][:, None, :]
            p = d[:, :, t[0]]
            for i in range(1, k):
                p = p * d[:, :, t[i]]
            return p
        out[k] = _reduce(unit, n_units, t.shape[1], product, total, 0.0)
    lo = hi = None
    if extrema:
        lo = _reduce(unit, n_units, m, plain, lambda t: t.amin(1), math.inf)
        hi = _reduce(unit, n_units, m, plain, lambda t: t.amax(1), -math.inf)
    return mean, out, lo, hi


def _exact_stats(c, cell, site_comp, comp_band, n_units, x):
    at, units = _units(cell, site_comp, comp_band)
    m, out = x.shape[0], {}
    diag = torch.tensor([j * m - j * (j - 1) // 2 for j in range(m)], device="cuda")
    for level, u, k in zip(("cell", "comp", "band"), units, n_units):
        mean, s, lo, hi = _centred(at, u, k, x, (2,), extrema=True)
        out[level] = {"n": None, "mean": mean, "m2": s[2][:, diag].contiguous(), "vmin": lo, "vmax": hi, "hist": None,
                      "cov": s[2] if c["cov"] else None}
    return out


def _neighbours(a, fill):
    """The six face neighbours' values of a volume."""
    for axis in range(3):
        n = a.shape[axis]
        for step in (1, -1):
            b = torch.full_like(a, fill)
            if n > 1:
                b.narrow(axis, 0 if step > 0 else 1, n - 1).copy_(a.narrow(axis, 1 if step > 0 else 0, n - 1))
            yield b


def _plain_lloyd(f, iso, seeds, iters):
    """Components, cells and mean displacements of a small uniform-weight step by synchronous sweeps in torch."""
    shape, n = f.shape, f.numel()
    band = sum((f > float(v)).int() for v in iso)
    lab = torch.arange(n, device="cuda").reshape(shape)
    edge = [b == band for b in _neighbours(band, -1)]
    while True:
        new = lab
        for e, b in zip(edge, _neighbours(lab, n)):
            new = torch.where(e, torch.minimum(new, b), new)
        new = new.reshape(-1)[new.reshape(-1)].reshape(shape)
        if torch.equal(new, lab):
            break
        lab = new
    first = torch.unique(lab)
    order = torch.argsort(band.reshape(-1)[first].long() * n + first)
    first = first[order]
    number = torch.empty(n, dtype=torch.long, device="cuda")
    number[first] = torch.arange(first.numel(), device="cuda")
    comp, comp_band = number[lab.reshape(-1)], band.reshape(-1)[first]
    far, hop = 1 << 62, 1 << 32
    sites, ds, ids = seeds.long(), [], torch.arange(seeds.numel(), device="cuda")
    idx = torch.arange(n, device="cuda")
    xyz = torch.stack([idx % shape[2], idx // shape[2] % shape[1], idx // (shape[2] * shape[1])])
    for k in range(iters + 1):
        key = torch.full((n,), far, device="cuda").scatter_reduce(0, sites, ids, "amin").reshape(shape)
        while True:
            new = key
            for e, b in zip(edge, _neighbours(key, far)):
                new = torch.where(e & (b < far), torch.minimum(new, b + hop), new)
            if torch.equal(new, key):
                break
            key = new
        cell = torch.where(key < far, key % hop, -1).reshape(-1)
        if k == iters:
            break
        at = torch.nonzero(cell >= 0).reshape(-1)
        u = cell[at]
        mass = torch.zeros_like(sites).index_add_(0, u, torch.ones_like(u))
        d = torch.zeros_like(u)
        for a in range(3):
            s = torch.zeros_like(sites).index_add_(0, u, xyz[a][at])
            d += (mass[u] * xyz[a][at] - s[u]) ** 2
        best = torch.full_like(sites, far).scatter_reduce(0, u, d * n + at, "amin")
        new = torch.where(mass > 0, best % n, sites)
        ds.append((xyz[:, new] - xyz[:, sites]).double().square().sum(0).sqrt().mean())
        sites = new
    return cell.int(), comp[seeds.long()], comp_band, first.numel(), torch.stack(ds) if ds else torch.zeros(0)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "step" and c["field"] == "blobs" and _voxels(c) <= 1 << 19:
        s = prepare(c, seed)
        cell, site_comp, comp_band, n_comp, ds = _plain_lloyd(s["f"], s["iso"], s["seeds"], c["iters"])
        n_units = (s["seeds"].numel(), n_comp, s["n_bands"])
        out = _exact_stats(c, cell, site_comp, comp_band, n_units, s["x"])
        return {"band": None, "status": None, "comp": None, "comp_band": None, "comp_size": None, "comp_first": None,
                "band_offset": None, "cells": None, "sites": None, "site_comp": None, "mean_ds": ds, **out}
    if kind not in ("stats", "moments", "layout"):
        return None  # whole numbers, or a loop that plain torch does not finish in the time
    s = prepare(c, seed)
    if kind == "layout":
        at, _ = _units(s["cell"], s["site_comp"], s["comp_band"])
        return {"perm": None, "site_order": None, "cell_off": None, "comp_off": None, "band_off": None,
                "raw": s["x"].reshape(s["x"].shape[0], -1)[:, at].double()}
    n_units = (s["sites"].numel(), s["n_comp"], s["n_bands"])
    if kind == "stats":
        return _exact_stats(c, s["cell"], s["site_comp"], s["comp_band"], n_units, s["x"])
    at, units = _units(s["cell"], s["site_comp"], s["comp_band"])
    out = {}
    for level, u, k in zip(("cell", "comp", "band"), units, n_units):
        mean, p, _, _ = _centred(at, u, k, s["x"], (2, 3, 4))
        out[level] = {"n": None, "mean": mean, "m2": p[2], "m3": p[3], "m4": p[4]}
    return out
