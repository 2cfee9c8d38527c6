"""The work this library is used for, as measurable cases.

A case is one call (or one step) through the public entry points on a
synthetic observation: Earth-rotation tracks of a random antenna layout,
time-major rows, a few per cent of flagged samples, noise-dominated
visibilities.  `kind` says which entry point it times:

  grid      lr_grid_overwrite with a resident plan (a major cycle's G)
  degrid    lr_degrid with a resident plan (a major cycle's D)
  psf       lr_make_psf with a resident plan
  job_*     the same calls without a plan: the one-off calls of a serving job
  stream    a plan build and an accumulating lr_grid, as a chunk streamed
            from host memory gets them
  chi2      value and image gradient of the weighted chi^2 (autograd)
  clean     a Hogbom minor cycle
"""

import math

import numpy as np
import torch

from paper_2508_17187_amd import lr
from paper_2508_17187_amd.autograd import DegridOp, chi2

C_LIGHT = 299792458.0
ARCSEC = math.pi / (180.0 * 3600.0)
LATITUDE = math.radians(34.0784)
DEC = math.radians(30.0)
OMEGA = 2.0 * math.pi / 86164.0905
DISH = 25.0
FLAGGED = 0.03


def _case(name, kind, precision, **kw):
    c = dict(name=name, kind=kind, precision=precision, n_ant=27, diameter_m=36000.0, n_time=600,
             dt_s=1.0 / 60.0, nchan=16, npol=4, n=2048, cell_arcsec=0.2, terms=3, oversample=20,
             n_w=32, h_min=8, h_max=32, n_fg=1, pointing=False, niter=0)
    c.update(kw)
    return c


PS = dict(terms=1, oversample=100, n_w=1, h_min=3, h_max=3)


def listed():
    return [
        # the smallest observation: one channel, one correlation, compact
        # array, Standard kernel, double precision; launches dominate
        _case("grid_plain_f64", "grid", "f64", diameter_m=1000.0, n_time=64, dt_s=56.25, nchan=1,
              npol=1, n=256, cell_arcsec=2.0, **PS),
        # a small serving job, inputs seen once: the call bins the samples itself
        _case("job_degrid_small_f32", "job_degrid", "f32", n_time=9, dt_s=10.0, nchan=5, n=512,
              cell_arcsec=0.2, n_w=11),
        # a serving job at the upper end of the stream's sizes
        _case("job_grid_f32", "job_grid", "f32", n_time=300, dt_s=0.5, nchan=12, npol=4, n=1024,
              cell_arcsec=0.2, n_w=48),
        # W-projection imaging, the gridding half of a major cycle
        _case("grid_wproj_f32", "grid", "f32"),
        # the same data in double precision
        _case("grid_wproj_f64", "grid", "f64"),
        # W-projection, the prediction half, kernels stored as FP16
        _case("degrid_wproj_f16cf", "degrid", "f16cf"),
        # the Standard kernel on the same data: bandwidth-bound
        _case("grid_ps_f32", "grid", "f32", **PS),
        # Standard kernel on a wide field: nearly every sample its own group
        _case("degrid_ps_wide_f32", "degrid", "f32", n_time=280, dt_s=2.0, nchan=64, n=8192,
              cell_arcsec=0.3, **PS),
        # a chunk of a large A+W image, both directions
        _case("grid_aw_large_f32", "grid", "f32", n_time=140, dt_s=2.0, nchan=64, n=8192,
              cell_arcsec=0.3, terms=7, n_w=128, h_max=64, n_fg=2),
        _case("degrid_aw_large_f32", "degrid", "f32", n_time=140, dt_s=2.0, nchan=64, n=8192,
              cell_arcsec=0.3, terms=7, n_w=128, h_max=64, n_fg=2),
        # A+W projection with per-antenna pointing offsets: one iteration of
        # an image solve (forward and backward)
        _case("chi2_aw_pointing_f32", "chi2", "f32", n_time=300, nchan=32, n=4096, terms=7, n_fg=4,
              pointing=True),
        # the minor cycle between two major cycles
        _case("clean_f32", "clean", "f32", n=2048, niter=100),
    ]


def draw(rng):
    """A case of the same ranges: 1e4 to 1.3e7 samples, 256 to 4096 pixels a
    side (8192 with the Standard kernel), every kernel family and storage."""
    kind = rng.choice(["grid", "grid", "degrid", "degrid", "psf", "job_grid", "job_degrid",
                       "stream"])
    precision = rng.choice(["f32", "f32", "f32", "f64", "f16cf", "bf16cf"])
    family = rng.choice(["ps", "w", "w", "aw"])
    npol = rng.choice([1, 2, 4, 4])
    nchan = int(round(2.0 ** rng.uniform(0.0, 6.0)))
    # kind and family bound the work: a pass stays below the largest listed one
    most = {"ps": 1.2e7, "w": 1.2e7, "aw": 5e6}[family]
    samples = 10.0 ** rng.uniform(4.0, math.log10(most))
    n_ant = rng.choice([15, 20, 27])
    n_time = max(4, int(samples / (n_ant * (n_ant - 1) // 2 * nchan * npol)))
    # odd multiples of 2 among the sizes: the sides need not be powers of two
    n = 2 * int(round(2.0 ** rng.uniform(7.0, 12.0 if family == "ps" else 11.0)))
    c = _case("", kind, precision, n_ant=n_ant, n_time=n_time, nchan=nchan, npol=npol, n=n,
              dt_s=rng.choice([1.0 / 60.0, 0.5, 2.0, 10.0]),
              # 0.2 arcsec keeps the longest baseline on the grid, 0.25 drops some
              cell_arcsec=rng.choice([0.2, 0.25]))
    if family == "ps":
        c.update(PS)
        c["h_min"] = c["h_max"] = rng.choice([3, 3, 4, 5])
    else:
        c.update(n_w=rng.randint(2, 64), oversample=rng.choice([8, 16, 20]),
                 h_min=rng.randint(3, 8), h_max=rng.randint(9, min(40, n // 16)),
                 terms=7 if family == "aw" else 3, n_fg=rng.randint(1, 3) if family == "aw" else 1)
        c["pointing"] = family == "aw" and kind in ("grid", "degrid") and rng.random() < 0.4
    c["n_fg"] = min(c["n_fg"], nchan)
    del c["name"]
    return c


# --- inputs -----------------------------------------------------------------

def _complex(case):
    return torch.complex128 if case["precision"] == "f64" else torch.complex64


def _real(case):
    return torch.float64 if case["precision"] == "f64" else torch.float32


def _layout(case, seed):
    """Coordinates and channel tables (host float64), pointing offsets."""
    rng = np.random.default_rng(seed)
    na, nt = case["n_ant"], case["n_time"]
    r = 0.5 * case["diameter_m"] * np.sqrt(rng.random(na))
    th = 2.0 * math.pi * rng.random(na)
    east, north = r * np.cos(th), r * np.sin(th)
    xyz = np.stack([-math.sin(LATITUDE) * north, east, math.cos(LATITUDE) * north], 1)
    a1, a2 = np.triu_indices(na, 1)
    bx, by, bz = (xyz[a2] - xyz[a1]).T
    ha = OMEGA * ((np.arange(nt) + 0.5) * case["dt_s"] - 0.5 * nt * case["dt_s"])[:, None]
    sh, ch, sd, cd = np.sin(ha), np.cos(ha), math.sin(DEC), math.cos(DEC)
    uvw = np.stack([sh * bx + ch * by, -sd * ch * bx + sd * sh * by + cd * bz,
                    cd * ch * bx - cd * sh * by + sd * bz], -1).reshape(-1, 3)
    nc = case["nchan"]
    freq = 2e9 + (np.arange(nc) + 0.5) * 2e9 / nc
    fg = (np.arange(nc) * case["n_fg"] // nc).astype(np.int32)
    fg_hz = np.array([freq[fg == g].mean() for g in range(case["n_fg"])])
    w_max = float(np.abs(uvw[:, 2]).max() * freq.max() / C_LIGHT) if case["n_w"] > 1 else 0.0
    dlm = rng.normal(0.0, 0.01 * 1.029 * (C_LIGHT / 3e9) / DISH, (na, 2))
    return dict(uvw=np.ascontiguousarray(uvw), freq=freq, fg=fg, fg_hz=fg_hz, w_max=w_max,
                ant1=np.tile(a1, nt).astype(np.int32), ant2=np.tile(a2, nt).astype(np.int32),
                dlm=dlm)


def _samples(case, seed, nrow):
    """Visibilities and weights (0: flagged), on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (nrow, case["nchan"], case["npol"])
    vis = torch.randn(shape, dtype=_complex(case), device="cuda", generator=g)
    wt = torch.rand(shape, dtype=_real(case), device="cuda", generator=g) + 0.5
    bad = torch.rand(shape[:2], device="cuda", generator=g) < FLAGGED
    wt[bad] = 0
    return vis, wt, g


def _model_grid(case, g):
    return torch.randn((1, case["npol"], case["n"], case["n"]), dtype=_complex(case),
                       device="cuda", generator=g)


def _model_image(case, g):
    """Two hundred point sources."""
    n, p = case["n"], case["npol"]
    img = torch.zeros((1, p, n, n), dtype=_real(case), device="cuda")
    yx = torch.randint(n // 8, n - n // 8, (2, 200), device="cuda", generator=g)
    for q in ((0, p - 1) if p > 1 else (0,)):
        img[0, q, yx[0], yx[1]] = torch.rand(200, dtype=_real(case), device="cuda", generator=g)
    return img


def _clean_inputs(case, seed):
    """A dirty image and its point-spread function: sources seen through the
    transfer function of random tracks, plus noise of the same coverage."""
    n = case["n"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    lay = _layout(dict(case, n_time=256, dt_s=60.0, diameter_m=30000.0), seed)
    uv = lay["uvw"][:, :2]
    px = torch.as_tensor(uv / np.abs(uv).max() * (0.4 * n), device="cuda").round().long()
    cover = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    for s in (1, -1):
        cover[(s * px[:, 1]) % n, (s * px[:, 0]) % n] = 1.0
    psf = torch.fft.ifft2(cover).real
    peak = psf[0, 0].clone()
    sky = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    yx = torch.randint(n // 4, 3 * n // 4, (2, 60), device="cuda", generator=g)
    sky[yx[0], yx[1]] = 0.1 + torch.rand(60, dtype=torch.float64, device="cuda", generator=g)
    noise = 1e-3 * n * torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    dirty = torch.fft.ifft2(cover * torch.fft.fft2(sky)).real / peak
    dirty = dirty + torch.fft.ifft2(cover * torch.fft.fft2(noise)).real
    dt = _real(case)
    return torch.fft.fftshift(psf / peak).to(dt).contiguous(), dirty.to(dt).contiguous()


def prepare(case, seed):
    p = lr.PRECISIONS[case["precision"]]
    n, npol, kind = case["n"], case["npol"], case["kind"]
    if kind == "clean":
        psf, dirty = _clean_inputs(case, seed)
        work = torch.empty(lr.lib().lr_hogbom_work_bytes(n, n), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, psf=psf, dirty=dirty, niter=case["niter"], work=work,
                    residual=torch.empty_like(dirty), model=torch.empty_like(dirty))
    lay = _layout(case, seed)
    cell = case["cell_arcsec"] * ARCSEC
    cf = lr.lr_cf_build(lr.GridSpec(n, n, npol, 1, cell, cell),
                        dict(terms=case["terms"], oversample=case["oversample"], ps_support=7,
                             n_w=case["n_w"], w_max=lay["w_max"], h_min=case["h_min"],
                             h_max=case["h_max"], n_fg=case["n_fg"], fg_hz=lay["fg_hz"],
                             dish_m=DISH, screen_m=0, storage=p, pol_beam=0, beam_ellipticity=0.0,
                             beam_leakage=0.0))
    vis, wt, g = _samples(case, seed, lay["uvw"].shape[0])
    po = {}
    if case["pointing"]:
        po = {k: torch.as_tensor(lay[s], device="cuda")
              for k, s in (("ant1", "ant1"), ("ant2", "ant2"), ("ant_dlm", "dlm"))}
    v = lr.Vis(torch.as_tensor(lay["uvw"], device="cuda"), lay["freq"], None, lay["fg"], vis=vis,
               weight=wt, npol=npol, **po)
    s = dict(kind=kind, p=p, cf=cf, v=v)
    if kind == "chi2":
        s.update(op=DegridOp(cf, v, p), image=_model_image(case, g).requires_grad_(True))
        return s
    back = kind.endswith("degrid")
    if not kind.startswith(("job", "stream")):
        s["v"] = v = v.with_(plan=lr.Plan(cf, v, psf=kind == "psf").packed())
    if kind == "stream":
        s["buf"] = torch.empty(lr.plan_bytes(cf, v), dtype=torch.uint8, device="cuda")
    op = lr.LR_OP_DEGRID if back else lr.LR_OP_PSF if kind == "psf" else lr.LR_OP_GRID
    s["work"] = torch.empty(lr.workspace_bytes(op, cf, v, p), dtype=torch.uint8, device="cuda")
    if back:
        s["v"] = v.with_(vis=torch.empty_like(vis))
        s["grid"] = _model_grid(case, g)
    else:
        s["grid"] = torch.empty((1, npol, n, n), dtype=_complex(case), device="cuda")
        s["sumwt"] = torch.empty((1, npol), dtype=torch.float64, device="cuda")
        s["counters"] = torch.empty(3, dtype=torch.int64, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "clean":
        s["residual"].copy_(s["dirty"])
        s["model"].zero_()
        it = lr.lr_hogbom(s["psf"], s["residual"], s["model"], 0.1, 0.0, s["niter"],
                          work=s["work"])
        return {"residual": s["residual"], "model": s["model"], "iterations": it}
    if kind == "chi2":
        value = chi2(s["image"], s["op"], s["v"].vis, s["v"].weight)
        grad, = torch.autograd.grad(value, s["image"])
        return {"chi2": value.detach(), "gradient": grad}
    cf, v, p = s["cf"], s["v"], s["p"]
    if kind.endswith("degrid"):
        lr.lr_degrid(cf, v, p, s["grid"], work=s["work"])
        return {"vis": v.vis}
    out = dict(sumwt=s["sumwt"], counters=s["counters"], work=s["work"])
    if kind in ("grid", "job_grid"):
        lr.lr_grid_overwrite(cf, v, p, s["grid"], **out)
    else:
        for t in (s["grid"], s["sumwt"], s["counters"]):
            t.zero_()
        if kind == "psf":
            lr.lr_make_psf(cf, v, p, s["grid"], **out)
        else:
            v = v.with_(plan=lr.Plan(cf, v, buf=s["buf"]))
            lr.lr_grid(cf, v, p, s["grid"], **out)
    return {"grid": s["grid"], "sumwt": s["sumwt"], "counters": s["counters"]}


# --- the same in 64 bits, in plain torch ------------------------------------

def _half_widths(case):
    d, m = case["h_max"] - case["h_min"], case["n_w"] - 1
    return [case["h_min"] + ((2 * d * k + m) // (2 * m) if m else 0) for k in range(m + 1)]


def _map(case, lay, psf=False):
    """Integer coordinates of every (row, channel): frequency group, w-plane,
    conjugation, pixel and offset on each axis, and whether it is kept."""
    n, o = case["n"], case["oversample"]
    cell = case["cell_arcsec"] * ARCSEC
    f = torch.as_tensor(lay["freq"], device="cuda")
    u, v, w = (torch.as_tensor(lay["uvw"][:, i].copy(), device="cuda")[:, None] for i in range(3))
    s = f / C_LIGHT
    at = [(x * (((s * n) * cell) * o) + (n // 2 * o + 0.5)) for x in (u, v)]
    k = torch.floor(w.abs() * (s * ((case["n_w"] - 1) / lay["w_max"])) + 0.5).long() \
        if case["n_w"] > 1 else torch.zeros_like(at[0], dtype=torch.long)
    keep = k < case["n_w"]
    k = k.clamp(max=case["n_w"] - 1)
    h = torch.as_tensor(_half_widths(case), device="cuda")[k]
    pix, off = [], []
    for x in at:
        q = torch.floor(x).long()
        c = (q + o // 2) // o
        keep &= (x >= 0) & (x < n * o) & (c - h >= (1 if psf else 0)) & (c + h <= n - 1)
        pix.append(c)
        off.append(q - c * o)
    fg = torch.as_tensor(lay["fg"], device="cuda").long().expand(k.shape)
    conj = (w < 0).expand(k.shape).long() if case["n_w"] > 1 else torch.zeros_like(k)
    return fg, k, conj, pix[1], pix[0], off[1], off[0], keep


def _groups(case, lay, psf=False):
    """Kept samples with the same kernel and footprint, merged: the group of
    every (row, channel) (-1: dropped) and each group's coordinates."""
    fg, k, conj, pv, pu, ov, ou, keep = _map(case, lay, psf)
    o, n = case["oversample"], case["n"]
    key = ((fg * case["n_w"] + k) * 2 + conj) * n + pv
    key = (key * n + pu) * o + (ov + o // 2)
    key = key * o + (ou + o // 2)
    if case["pointing"]:
        na, nc = case["n_ant"], case["nchan"]
        bl = torch.as_tensor(lay["ant1"].astype(np.int64) * na + lay["ant2"], device="cuda")
        # both parts are compacted first so that the combined key fits 63 bits
        _, key = torch.unique(key.reshape(-1), return_inverse=True)
        key = key.reshape(k.shape) * (na * na * nc) + (bl[:, None] * nc +
                                                       torch.arange(nc, device="cuda"))
    key = torch.where(keep, key, torch.full_like(key, -1)).reshape(-1)
    uniq, group = torch.unique(key, return_inverse=True)
    if uniq[0] < 0:
        group = group - 1
    n_groups = int(uniq.numel()) - int(uniq[0] < 0)
    first = torch.full((n_groups,), key.numel(), dtype=torch.long, device="cuda")
    idx = torch.nonzero(group >= 0)[:, 0]
    first.scatter_reduce_(0, group[idx], idx, "amin")
    cols = {c: t.reshape(-1)[first] for c, t in
            (("fg", fg), ("k", k), ("conj", conj), ("pv", pv), ("pu", pu), ("ov", ov), ("ou", ou))}
    if case["pointing"]:
        nc = case["nchan"]
        row, ch = first // nc, first % nc
        d = torch.as_tensor(lay["dlm"], device="cuda")
        d1 = d[torch.as_tensor(lay["ant1"], device="cuda").long()[row]]
        d2 = d[torch.as_tensor(lay["ant2"], device="cuda").long()[row]]
        nu = torch.as_tensor(lay["freq"], device="cuda")[ch]
        cols["shift"] = 0.5 * (d1 + d2)
        cols["loss"] = _airy(math.pi * DISH * nu / C_LIGHT * 0.5 * (d1 - d2).norm(dim=1))
    return group, cols


def _airy(x):
    y = torch.where(x == 0, torch.ones_like(x), x)
    return torch.where(x == 0, torch.ones_like(x), (2 * torch.special.bessel_j1(y) / y) ** 2)


def _taper(x):
    """Prolate spheroidal psi_0(7 pi / 2, x), psi_0(0) = 1: the leading
    eigenfunction of the finite cosine transform on Gauss-Legendre nodes."""
    c = 3.5 * math.pi
    t, w = np.polynomial.legendre.leggauss(64)
    vec = np.linalg.eigh(np.sqrt(w)[:, None] * np.cos(c * np.outer(t, t)) * np.sqrt(w))[1][:, -1]
    y = np.cos(c * np.outer(x, t)) @ (np.sqrt(w) * vec)
    return y / (np.sqrt(w) @ vec)


def _kernel_plane(case, lay, fg, k):
    """[O+1][O+1][S][S] kernels of one plane."""
    hs = _half_widths(case)
    m, o, h = 2 * (2 * max(hs) + 1), case["oversample"], hs[k]
    width = case["n"] * case["cell_arcsec"] * ARCSEC
    j = np.arange(-(m // 2), m // 2 + 1)
    l = j * width / m
    edge = np.ones(m + 1)
    edge[0] = edge[-1] = 0.5
    tap = edge * (_taper(2 * l / width) if case["terms"] & 1 else 1.0)
    l, tap = torch.as_tensor(l, device="cuda"), torch.as_tensor(tap, device="cuda")
    r2 = l[:, None] ** 2 + l[None, :] ** 2
    screen = (tap[:, None] * tap[None, :]).to(torch.complex128)
    if case["terms"] & 4:
        screen = screen * _airy(math.pi * DISH * float(lay["fg_hz"][fg]) / C_LIGHT * r2.sqrt())
    if case["terms"] & 2 and k:
        n1 = -r2 / (1 + (1 - r2).clamp(min=0).sqrt())
        wk = k * lay["w_max"] / (case["n_w"] - 1)
        screen = torch.where(r2 < 1, screen * torch.polar(torch.ones_like(n1),
                                                          -2 * math.pi * wk * n1), 0 * screen)
    at = np.arange(-(o // 2), o // 2 + 1)[:, None] - o * np.arange(-h, h + 1)[None, :]
    ph = (np.outer(at.ravel(), j) % (o * m)) * (-2 * math.pi / (o * m))
    e = torch.polar(torch.ones(ph.shape, dtype=torch.float64), torch.as_tensor(ph)).cuda()
    kern = (e @ screen @ e.T) / (m * m)
    return kern.reshape(o + 1, 2 * h + 1, o + 1, 2 * h + 1).permute(0, 2, 1, 3).conj().resolve_conj()


def _batches(case, lay, cols, most=6_000_000):
    """(groups, kernels [g][S][S], cells [g][S][S]) of bounded size."""
    n, o, hs = case["n"], case["oversample"], _half_widths(case)
    cell = case["cell_arcsec"] * ARCSEC
    plane = cols["fg"] * case["n_w"] + cols["k"]
    order = torch.argsort(plane)
    ids, counts = torch.unique_consecutive(plane[order], return_counts=True)
    at = 0
    for i, c in zip(ids.tolist(), counts.tolist()):
        fg, k = divmod(i, case["n_w"])
        h = hs[k]
        size = 2 * h + 1
        table = _kernel_plane(case, lay, fg, k).reshape(-1, size, size)
        t = torch.arange(-h, h + 1, device="cuda")
        for g in order[at:at + c].split(max(1, most // size ** 2)):
            ker = table[(cols["ov"][g] + o // 2) * (o + 1) + cols["ou"][g] + o // 2]
            ker = torch.where(cols["conj"][g].bool()[:, None, None], ker.conj(), ker)
            if case["pointing"]:
                # exp(-2 pi i (t - o / O) . shift / (n cell)) on each axis
                ph = [((t - cols[a][g][:, None] / o) * (cols["shift"][g, x:x + 1] / (n * cell)))
                      for a, x in (("ov", 1), ("ou", 0))]
                ph = -2 * math.pi * (ph[0][:, :, None] + ph[1][:, None, :])
                ker = ker * torch.polar(cols["loss"][g][:, None, None].expand(ph.shape), ph)
            cells = (cols["pv"][g][:, None, None] + t[:, None]) * n + (cols["pu"][g][:, None, None]
                                                                     + t)
            yield g, ker, cells
        at += c


def _exact_grid(case, lay, group, cols, sums):
    """grid [npol][n * n] of the group sums [groups][npol]."""
    n = case["n"]
    out = torch.zeros((case["npol"], n * n, 2), dtype=torch.float64, device="cuda")
    for g, ker, cells in _batches(case, lay, cols):
        cells = cells.reshape(-1)
        for q in range(case["npol"]):
            val = torch.view_as_real(ker * sums[g, q][:, None, None]).reshape(-1, 2)
            out[q].index_add_(0, cells, val)
    return torch.view_as_complex(out).reshape(1, case["npol"], n, n)


def _exact_degrid(case, lay, group, cols, grid):
    """[groups][npol] of a grid [1][npol][n][n]."""
    flat = grid.reshape(case["npol"], -1)
    out = torch.zeros((cols["k"].numel(), case["npol"]), dtype=torch.complex128, device="cuda")
    for g, ker, cells in _batches(case, lay, cols):
        for q in range(case["npol"]):
            out[g, q] = (ker.conj() * flat[q][cells]).sum((1, 2))
    return out


def _centred_fft2(img):
    return torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(img, dim=(-2, -1))), dim=(-2, -1))


def exact(case, seed):
    kind = case["kind"]
    if kind == "clean":
        # a sequence of choices of the largest pixel: rounding may swap two
        # near-equal ones, so no value at higher precision is "the" result
        return None
    lay = _layout(case, seed)
    vis, wt, g = _samples(case, seed, lay["uvw"].shape[0])
    group, cols = _groups(case, lay, kind == "psf")
    npol, n_groups = case["npol"], cols["k"].numel()
    pairs = torch.nonzero(group >= 0)[:, 0]
    member = group[pairs]

    def sums(values):
        a = torch.zeros((n_groups, npol, 2), dtype=torch.float64, device="cuda")
        a.index_add_(0, member, torch.view_as_real(values.reshape(-1, npol)[pairs]))
        return torch.view_as_complex(a)

    def spread(values):
        out = torch.zeros((group.numel(), npol), dtype=torch.complex128, device="cuda")
        out[pairs] = values[member]
        return out.reshape(vis.shape) * (wt != 0)

    if kind == "chi2":
        img = _model_image(case, g).double().requires_grad_(True)
        grid = _centred_fft2(img.to(torch.complex128))
        model = spread(_exact_degrid(case, lay, group, cols, grid.detach()))
        r = vis.to(torch.complex128) - model
        value = (wt.double() * (r.real ** 2 + r.imag ** 2)).sum()
        back = _exact_grid(case, lay, group, cols, sums((-2.0 * wt) * r * (wt != 0)))
        grad, = torch.autograd.grad(grid, img, back)
        return {"chi2": value, "gradient": grad}
    if kind.endswith("degrid"):
        grid = _model_grid(case, g).to(torch.complex128)
        return {"vis": spread(_exact_degrid(case, lay, group, cols, grid))}
    w = wt.double()
    unit = torch.ones_like(vis) if kind == "psf" else vis
    out = _exact_grid(case, lay, group, cols, sums(w * unit.to(torch.complex128)))
    if kind == "psf":
        mirror = torch.roll(out.flip((-2, -1)), (1, 1), (-2, -1)).conj()
        out = 0.5 * (out + mirror)
    kept = w.reshape(-1, npol)[pairs]
    n_kept, n_flagged = int((kept != 0).sum()), int((w == 0).sum())
    return {"grid": out, "sumwt": kept.sum(0, keepdim=True),
            "counters": torch.tensor([n_kept, n_flagged, w.numel() - n_kept - n_flagged])}


def work(case):
    """Bytes: samples in or out once, the grid once, and the kernels that the
    samples meet once (an even screen makes the kernels of offsets o and -o
    mirror images, so one of them determines both).  Flops: one complex
    multiply-add per tap and correlation of the merged samples (real kernels
    half of that)."""
    n, npol, kind = case["n"], case["npol"], case["kind"]
    size = {"f64": 8}.get(case["precision"], 4)
    if kind == "clean":
        # every subtraction reads the image and the point-spread function
        # and writes the image
        return {"bytes": 3.0 * size * n * n * case["niter"], "flops": 2.0 * n * n * case["niter"]}
    elem = {"f64": 16, "f32": 8}.get(case["precision"], 4)
    group, cols = _groups(case, _layout(case, 1), kind == "psf")
    side = 2 * torch.as_tensor(_half_widths(case), device="cuda") + 1
    o = case["oversample"]
    off = (cols["fg"] * case["n_w"] + cols["k"]) * (o + 1) + cols["ov"].abs()
    kernels = torch.unique(off * (o + 1) + cols["ou"].abs()) // ((o + 1) * (o + 1))
    table = elem * float((side[kernels % case["n_w"]] ** 2).sum())
    if case["terms"] == 1:
        table = elem * (o + 1) * float(side[0])        # outer products of one row
    taps = float((side[cols["k"]] ** 2).sum())
    samples = float(group.numel()) * npol
    io = {"psf": size, "degrid": 3 * size, "job_degrid": 3 * size}.get(kind, 3 * size)
    passes = 2 if kind == "chi2" else 1
    b = samples * io + 2.0 * size * npol * n * n + table
    if kind.startswith(("job", "stream")):
        b += 24.0 * group.numel() / case["nchan"]
    f = taps * npol * (4.0 if case["terms"] == 1 else 8.0)
    if kind == "chi2":
        # forward and backward transforms of the image
        f += 2 * 5.0 * n * n * npol * math.log2(float(n) * n) / passes
    return {"bytes": passes * b, "flops": passes * f}
