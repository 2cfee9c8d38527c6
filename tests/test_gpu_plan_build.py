"""GPU: the binning plan at the edges of its passes: tiles holding one pair
less than, exactly and one more than whole gridder chunks, plans in which
every pair, the last pair or no pair is kept, keys too wide to merge
groups, and sort sizes on both sides of the merge sort's limit.  Counts
against the oracle's index map, the grid against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from oracle.cfbuild import TERM_A, TERM_PS, TERM_W
from oracle.native import Problem
from synth.observation import C_LIGHT

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_17187_amd import lr  # noqa: E402
from paper_2508_17187_amd import workload as W  # noqa: E402


def lattice(n, wide=False, nx=96):
    """n samples, each its own group, the first 1000 of them footprints of
    one 32 x 32 tile, later ones anywhere on the grid (some dropped)."""
    o = 8 if not wide else 126
    kw = dict(n_ant=4, n_time=max(1, -(-n // 6)), nchan=1, npol=1, nx=nx, ny=nx, cell_arcsec=6.0,
              oversample=o, terms=TERM_PS, cfg_id=270)
    if wide:
        kw.update(terms=TERM_PS | TERM_W | TERM_A, n_w=4, h_min=2, h_max=3, pointing_sigma=3e-5)
    wl = synth.tiny_workload(**kw)
    rng = np.random.default_rng(n)
    m = wl.obs.nrow
    du = 1.0 / (nx * wl.grid.cell_l) * C_LIGHT / wl.obs.freq_hz[0]     # metres per cell
    i = np.arange(m)
    x = np.where(i < n, 40 + (i % 16) + 0.3 + (i // 256 % 4) / o, 1e4)
    y = 40 + (i // 16 % 16) + 0.3 + (i // 1024) / o
    far = (i >= 1000) & (i < n)
    x[far], y[far] = rng.uniform(0, nx, far.sum()), rng.uniform(0, nx, far.sum())
    wl.obs.uvw[:, 0] = (x - nx // 2) * du
    wl.obs.uvw[:, 1] = (y - nx // 2) * du
    if not wide:
        wl.obs.uvw[:, 2] = 0.0
    return wl


def check(wl, precision=lr.LR_F64):
    cf = W.build_cf(wl, precision)
    v = W.device_vis(wl, precision)
    pr = Problem.from_workload(wl, oracle.build_cf(wl.grid, wl.cf))
    plan = lr.Plan(cf, v)
    info = plan.info()
    m = lr.lr_debug_map(cf, v).cpu().numpy().reshape(-1, 8)
    on = np.tile(np.asarray(wl.chan_plane) >= 0, wl.obs.nrow)       # the map ignores planes
    kept = m[(m[:, 6] == 1) & on]
    assert info["n_kept"] == len(kept) and info["n_pairs"] == len(m)
    ref = pr.grid(wl.vis, wl.weight)
    for plan_ in (plan, plan.packed(), None):
        g = W.empty_grid(wl, precision)
        c = torch.zeros(3, dtype=torch.int64, device="cuda")
        lr.lr_grid(cf, v.with_(plan=plan_), precision, g, counters=c)
        # FP64 parity bound of the library
        assert np.linalg.norm(g.cpu().numpy() - ref) <= 1e-12 * max(np.linalg.norm(ref), 1e-300)
        assert c.cpu().numpy()[0] == len(kept) * wl.grid.npol
    return info, kept


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 1000, 5000, 32767, 32768, 32769,
                               40000, 262143, 262144, 262150])
def test_chunk_edges(n):
    info, kept = check(lattice(n))
    assert info["n_groups"] == len(np.unique(kept[:, :6], axis=0))
    assert info["taps"] == 49 * info["n_groups"]


@pytest.mark.parametrize("h", [1, 3, 4, 6, 7])
@pytest.mark.parametrize("form", ["f64", "f32"])
def test_few_tiles_in_many_parts(h, form):
    """Dense data on few tiles: the separable gridder's tiles are cut into
    parts that add to shared tiles, accumulating and overwriting."""
    prec = lr.PRECISIONS[form]
    wl = synth.tiny_workload(n_ant=9, n_time=150, dt_s=90.0, nchan=3, npol=2, nx=160, ny=100,
                             cell_arcsec=20.0, diameter_m=1500.0, oversample=32, terms=TERM_PS,
                             h_min=h, h_max=h, cfg_id=273)
    cf = W.build_cf(wl, prec)
    v = W.device_vis(wl, prec)
    v.plan = lr.Plan(cf, v)
    ref = Problem.from_workload(wl, oracle.build_cf(wl.grid, wl.cf)).grid(wl.vis, wl.weight)
    tol = {"f64": 1e-12, "f32": 1e-5}[form] * np.linalg.norm(ref)
    g = W.empty_grid(wl, prec)
    lr.lr_grid(cf, v, prec, g)
    assert np.linalg.norm(g.cpu().numpy() - ref) <= tol
    g.fill_(complex("nan"))
    lr.lr_grid_overwrite(cf, v, prec, g)
    assert np.linalg.norm(g.cpu().numpy() - ref) <= tol


@pytest.mark.parametrize("nx,n", [(2048, 1100), (4096, 5000), (4096, 7000), (8192, 22000)])
def test_parts_do_not_depend_on_the_empty_tiles(nx, n):
    """The same samples around the centre of a large grid and of a 256^2 one
    with the same cells: four tiles hold them all, and the packed plans
    differ by their per-tile arrays alone, so both are cut into as many
    parts; the grids agree (FP64 rounding of another order of additions)."""
    plans, grids = [], []
    for side in (256, nx):
        wl = synth.tiny_workload(n_ant=4, n_time=-(-n // 6), nchan=1, npol=1, nx=side, ny=side,
                                 cell_arcsec=6.0 * 256 / side, oversample=20, terms=TERM_PS,
                                 cfg_id=274)
        rng = np.random.default_rng(n)
        wl.obs.uvw[:] = 0.0
        wl.obs.uvw[:, :2] = rng.uniform(-28, 28, (wl.obs.nrow, 2)) / \
            (side * wl.grid.cell_l) * C_LIGHT / wl.obs.freq_hz[0]
        cf = W.build_cf(wl, lr.LR_F64)
        v = W.device_vis(wl, lr.LR_F64)
        plan = lr.Plan(cf, v)
        assert plan.info()["n_kept"] == wl.obs.nrow
        plans.append(plan.packed().buf.numel())
        g = W.empty_grid(wl, lr.LR_F64)
        lr.lr_grid(cf, v.with_(plan=plan), lr.LR_F64, g)
        lo = side // 2 - 128
        grids.append(g[..., lo:lo + 256, lo:lo + 256])
    aligned = lambda words: -(-4 * words // 256) * 256                  # noqa: E731
    tiles = [(side // 32) ** 2 for side in (256, nx)]
    per_tile = [aligned(t) + aligned(t + 1) for t in tiles]
    assert plans[1] - plans[0] == per_tile[1] - per_tile[0]
    assert (grids[1] - grids[0]).abs().max() <= 1e-12 * grids[0].abs().max()


def test_no_pair_kept():
    wl = lattice(6)
    wl.obs.uvw[:, 0] = 1e6
    info, kept = check(wl)
    assert info["n_groups"] == info["taps"] == len(kept) == 0


def test_every_pair_kept_with_a_skipped_channel():
    wl = synth.tiny_workload(nchan=4, chan_plane=[0, -1, 1, 0], nplane=2, cfg_id=271)
    info, kept = check(wl)
    assert info["n_kept"] < info["n_pairs"]
    wl = synth.tiny_workload(nchan=1, diameter_m=500.0, cfg_id=272)
    info, kept = check(wl)
    assert info["n_kept"] == info["n_pairs"]


@pytest.mark.parametrize("n", [130, 1500])
def test_wide_keys(n):
    """Baseline, channel and offset fields of an oversampling of 126."""
    check(lattice(n, wide=True))
