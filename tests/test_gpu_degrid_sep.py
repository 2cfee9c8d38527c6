"""GPU: degridding through single-plane real tables (the Standard kernel) at
every support the 32-lane kernel takes and the first it does not, in each
FP32 form and number of correlations: footprints starting at odd and even
columns, mirrored on each axis, at the grid's edges, group counts that leave
part of a wavefront or workgroup idle; cubes and FP64, which take the other
kernels."""

import numpy as np
import pytest

import oracle
import synth
from oracle.cfbuild import TERM_A, TERM_PS, quantised_table
from oracle.native import Problem
from synth.observation import C_LIGHT

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_17187_amd import lr  # noqa: E402
from paper_2508_17187_amd import workload as W  # noqa: E402

STORE = {"f64": "f64", "f32": "f32", "f16cf": "f16", "bf16cf": "bf16"}
# against the table as the form stores it: sums of 225 products of either sign
# in FP32, each of relative error 2^-24, and FP64 at the library's bound
TOL = {"f64": 1e-12, "f32": 1e-6, "f16cf": 1e-6, "bf16cf": 1e-6}


def degrid(form, h, npol, n_time, nplane=1):
    prec = lr.PRECISIONS[form]
    wl = synth.tiny_workload(n_ant=6, n_time=n_time, nchan=2, npol=npol, nx=74, ny=60,
                             cell_arcsec=6.0, diameter_m=3500.0, oversample=10, terms=TERM_PS,
                             h_min=h, h_max=h, nplane=nplane,
                             chan_plane=[0, nplane - 1], cfg_id=290)
    rng = np.random.default_rng(290 + h)
    wl.obs.uvw[:, :2] += rng.normal(0.0, 30.0, wl.obs.uvw[:, :2].shape)
    shape = (nplane, npol, 60, 74)
    g = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    cf = W.build_cf(wl, prec)
    v = W.device_vis(wl, prec)
    v.plan = lr.Plan(cf, v)
    lr.lr_degrid(cf, v, prec, torch.as_tensor(g, device="cuda").to(v.vis.dtype))
    ocf = oracle.build_cf(wl.grid, wl.cf)
    pr = Problem.from_workload(wl, ocf, table=quantised_table(ocf, STORE[form]))
    return v.vis.cpu().numpy(), pr.degrid(g.astype(np.complex128), wl.weight)


@pytest.mark.parametrize("form", ["f32", "f16cf", "bf16cf"])
@pytest.mark.parametrize("npol", [1, 2, 4])
@pytest.mark.parametrize("h", [0, 1, 2, 3, 4, 5, 7, 8])
def test_every_support(form, npol, h):
    got, ref = degrid(form, h, npol, 40)
    assert np.linalg.norm(got - ref) <= TOL[form] * np.linalg.norm(ref)


@pytest.mark.parametrize("n_time", [1, 2, 3, 7, 33, 270])
def test_group_counts(n_time):
    got, ref = degrid("f32", 3, 4, n_time)
    assert np.linalg.norm(got - ref) <= TOL["f32"] * np.linalg.norm(ref)


@pytest.mark.parametrize("form,nplane", [("f64", 1), ("f32", 3)])
def test_other_kernels(form, nplane):
    got, ref = degrid(form, 3, 4, 40, nplane)
    assert np.linalg.norm(got - ref) <= TOL[form] * np.linalg.norm(ref)


@pytest.mark.parametrize("form", ["f32", "f16cf"])
@pytest.mark.parametrize("npol", [1, 4])
@pytest.mark.parametrize("terms", [TERM_PS, TERM_PS | TERM_A])
@pytest.mark.parametrize("h", [8, 20, 31, 32, 62, 63, 64, 65, 128])
def test_pairs_per_row_around_a_wavefront(form, npol, terms, h):
    """Wider supports, real and complex: rows of 9 to 129 pairs on the 64
    lanes, on both sides of one and of two rows per step.  Against the stored
    table, at the library's FP32 bound (each lane adds up to 1000 products)."""
    prec = lr.PRECISIONS[form]
    wl = synth.tiny_workload(n_ant=4, n_time=40, nchan=1, npol=npol, nx=2 * h + 38, ny=2 * h + 30,
                             cell_arcsec=6.0, oversample=4, terms=terms, h_min=h, h_max=h,
                             fg_hz=[3e9], cfg_id=292)
    rng = np.random.default_rng(292 + h)
    wl.obs.uvw[:, :2] = rng.uniform(-14, 14, (wl.obs.nrow, 2)) / \
        ((2 * h + 38) * wl.grid.cell_l) * C_LIGHT / wl.obs.freq_hz[0]
    shape = (1, npol, 2 * h + 30, 2 * h + 38)
    g = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    cf = W.build_cf(wl, prec)
    v = W.device_vis(wl, prec)
    m = lr.lr_debug_map(cf, v).cpu().numpy()[:, 0]
    # odd and even starts, mirrored and not on each axis
    assert len({(a % 2, b > 0, c > 0) for a, b, c, k in m[:, [0, 2, 3, 6]] if k}) == 8
    lr.lr_degrid(cf, v, prec, torch.as_tensor(g, device="cuda"))
    ocf = oracle.build_cf(wl.grid, wl.cf)
    pr = Problem.from_workload(wl, ocf, table=quantised_table(ocf, STORE[form]))
    ref = pr.degrid(g.astype(np.complex128), wl.weight)
    assert np.linalg.norm(v.vis.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("form", ["f64", "f32", "f16cf", "bf16cf"])
@pytest.mark.parametrize("npol", [1, 4])
@pytest.mark.parametrize("h", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_cells_outside_a_footprint_are_not_read_into_it(form, npol, h, bad):
    """Every cell but one footprint's holds a value that is not finite: the
    footprint's sample is what zeros there give, bit for bit, whether it
    begins at an odd or an even column, mirrored or not."""
    prec = lr.PRECISIONS[form]
    wl = synth.tiny_workload(n_ant=6, n_time=30, nchan=1, npol=npol, nx=74, ny=60,
                             cell_arcsec=6.0, diameter_m=3500.0, oversample=10, terms=TERM_PS,
                             h_min=h, h_max=h, cfg_id=291)
    rng = np.random.default_rng(291 + h)
    wl.obs.uvw[:, :2] += rng.normal(0.0, 30.0, wl.obs.uvw[:, :2].shape)
    cf = W.build_cf(wl, prec)
    v = W.device_vis(wl, prec)
    v.plan = lr.Plan(cf, v)
    v.weight.fill_(1.0)
    m = lr.lr_debug_map(cf, v).cpu().numpy()[:, 0]
    shape = (1, npol, 60, 74)
    g = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    g = torch.as_tensor(g, device="cuda").to(v.vis.dtype)
    for odd in (0, 1):
        for side in (-1, 1):
            rows = np.nonzero((m[:, 6] == 1) & ((m[:, 0] - h) % 2 == odd) &
                              (np.where(m[:, 2] > 0, 1, -1) == side))[0]
            for row in rows[:3]:
                pu, pv = m[row, :2]
                out = []
                for fill in (0.0, bad):
                    q = torch.full_like(g, complex(fill, fill))
                    cut = np.s_[..., pv - h:pv + h + 1, pu - h:pu + h + 1]
                    q[cut] = g[cut]
                    lr.lr_degrid(cf, v, prec, q)
                    out.append(v.vis[row, 0].cpu().numpy().copy())
                assert np.isfinite(out[1]).all() and np.array_equal(out[0], out[1])
            assert len(rows)
