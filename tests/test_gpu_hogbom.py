"""GPU: Hogbom minor cycle (lr_hogbom) against the oracle's loop.

FP64 is compared bit for bit (the same operations in the same order and the
same tie rule give the same components); FP32 within rounding."""

import numpy as np
import pytest

import synth
import oracle
from oracle.cfbuild import TERM_PS
from oracle.hogbom import hogbom
from oracle.imaging import centred_ifft, gcf_1d, separable_1d
from oracle.native import Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_17187_amd import lr  # noqa: E402

DEV = "cuda"


@pytest.fixture(scope="module")
def dirty_and_psf():
    """Dirty image and PSF of a small point-source observation, made by the
    oracle (Stokes I plane)."""
    wl = synth.tiny_workload(n_ant=10, n_time=40, dt_s=300.0, nchan=2, nx=96, ny=96,
                             cell_arcsec=6.0, oversample=20, terms=TERM_PS, n_src=4,
                             sigma=0.002, cfg_id=99)
    ocf = oracle.build_cf(wl.grid, wl.cf)
    pr = Problem.from_workload(wl, ocf)
    c1 = separable_1d(ocf)
    gx = gcf_1d(c1, ocf.O, wl.grid.nx).real
    gy = gcf_1d(c1, ocf.O, wl.grid.ny).real
    corr = np.outer(gy, gx)
    s, _ = pr.sumwt(wl.weight)
    dirty = centred_ifft(pr.grid(wl.vis, wl.weight))[0, 0].real / corr / s[0, 0]
    psfg, s2, _ = pr.psf(wl.weight)
    psf = centred_ifft(psfg)[0, 0].real / corr / s2[0, 0]
    return np.ascontiguousarray(dirty), np.ascontiguousarray(psf)


def run(dirty, psf, dtype, gain, threshold, niter):
    res = torch.as_tensor(dirty, dtype=dtype, device=DEV).contiguous()
    p = torch.as_tensor(psf, dtype=dtype, device=DEV).contiguous()
    model = torch.zeros_like(res)
    it = lr.lr_hogbom(p, res, model, gain, threshold, niter)
    return model.cpu().numpy(), res.cpu().numpy(), it


def test_fp64_identical_to_oracle(dirty_and_psf):
    dirty, psf = dirty_and_psf
    thr = 0.02 * np.max(np.abs(dirty))
    m_ref, r_ref, it_ref = hogbom(dirty, psf, 0.1, thr, 400)
    m, r, it = run(dirty, psf, torch.float64, 0.1, thr, 400)
    print("hogbom iterations", it, it_ref, flush=True)
    assert it == it_ref and it > 20
    assert np.array_equal(m, m_ref)
    assert np.array_equal(r, r_ref)


def test_fp32_within_rounding(dirty_and_psf):
    dirty, psf = dirty_and_psf
    thr = 0.05 * np.max(np.abs(dirty))
    m_ref, r_ref, it_ref = hogbom(dirty, psf, 0.1, thr, 200)
    m, r, it = run(dirty, psf, torch.float32, 0.1, thr, 200)
    assert abs(it - it_ref) <= 2
    assert abs(m.sum() - m_ref.sum()) <= 1e-3 * abs(m_ref.sum())
    assert np.max(np.abs(r - r_ref)) <= 2e-2 * np.max(np.abs(dirty))


def test_budget_threshold_and_argument_checks(dirty_and_psf):
    dirty, psf = dirty_and_psf
    m, r, it = run(dirty, psf, torch.float64, 0.1, 0.0, 0)
    assert it == 0 and not m.any() and np.array_equal(r, dirty)
    m, r, it = run(dirty, psf, torch.float64, 0.1, 2 * np.max(np.abs(dirty)), 100)
    assert it == 0 and not m.any()
    m, r, it = run(dirty, psf, torch.float64, 1.0, 0.0, 1)
    assert it == 1 and np.count_nonzero(m) == 1
    with pytest.raises(lr.LRError) as ei:
        run(dirty, psf, torch.float64, 0.0, 0.0, 10)
    assert ei.value.status == lr.LR_E_ARG


def test_ragged_image_and_ties():
    """Odd sizes (centre at (ny/2, nx/2) with integer division) and an exact
    tie between two peaks: the lower index is cleaned first on both sides."""
    ny, nx = 37, 52
    rng = np.random.default_rng(11)
    psf = np.zeros((ny, nx))
    psf[ny // 2 - 2:ny // 2 + 3, nx // 2 - 3:nx // 2 + 4] = rng.uniform(0.1, 0.5, (5, 7))
    psf[ny // 2, nx // 2] = 1.0
    dirty = rng.normal(0, 0.01, (ny, nx))
    dirty[3, 50] = 1.0
    dirty[30, 2] = -1.0
    m_ref, r_ref, it_ref = hogbom(dirty, psf, 0.3, 0.05, 60)
    m, r, it = run(dirty, psf, torch.float64, 0.3, 0.05, 60)
    assert it == it_ref
    assert np.array_equal(m, m_ref) and np.array_equal(r, r_ref)


@pytest.mark.parametrize("ny,nx", [(1, 1), (3, 2), (5, 3), (37, 50), (64, 1023), (600, 1001),
                                   (1500, 1400)])
@pytest.mark.parametrize("niter", [1, 2, 9])
def test_sizes_around_the_quads_and_workgroups(ny, nx, niter):
    """Rows that are not whole quads of pixels, images smaller than a
    workgroup and larger than one pass of all of them, peaks near the edges
    (the PSF partly outside on each side): identical to the oracle in FP64."""
    rng = np.random.default_rng(ny * nx)
    psf = rng.normal(0, 0.1, (ny, nx))
    psf[ny // 2, nx // 2] = 1.0
    dirty = rng.normal(0, 0.1, (ny, nx))
    for y, x, v in ((0, 0, 3.0), (ny - 1, nx - 1, -2.9), (ny // 2, nx - 1, 2.8)):
        dirty[y, x] = v
    m_ref, r_ref, it_ref = hogbom(dirty, psf, 0.2, 0.0, niter)
    m, r, it = run(dirty, psf, torch.float64, 0.2, 0.0, niter)
    assert it == it_ref
    assert np.array_equal(m, m_ref) and np.array_equal(r, r_ref)


def test_no_finite_pixel_and_reuse_of_the_workspace():
    res = torch.full((40, 40), float("nan"), dtype=torch.float64, device=DEV)
    psf, model = torch.ones_like(res), torch.zeros_like(res)
    work = torch.full((lr.lib().lr_hogbom_work_bytes(40, 40),), 0x7F, dtype=torch.uint8, device=DEV)
    assert lr.lr_hogbom(psf, res, model, 0.1, 0.0, 5, work=work) == 0
    assert not model.any()
    res = torch.zeros_like(res)
    res[7, 9] = 1.0
    assert lr.lr_hogbom(psf, res, model, 0.1, 0.5, 3, work=work) == 3
    assert model.count_nonzero() == 1 and model[7, 9] != 0


@pytest.mark.parametrize("ny,nx", [(30, 40), (700, 1001)])
def test_exit_long_before_the_budget(ny, nx):
    """The exit test met after 0 to a few launches of 300, on one and on many
    workgroups: no workgroup of that launch or of a later one subtracts
    anything, whatever values the launches before left in its LDS."""
    rng = np.random.default_rng(ny)
    psf = rng.normal(0, 0.01, (ny, nx))
    psf[ny // 2, nx // 2] = 1.0
    dirty = rng.uniform(-0.01, 0.01, (ny, nx))
    for k in range(6):
        dirty[5 * k + 2, 6 * k + 3] = 10.0 * (6 - k)
    for rep in range(8):
        for thr in (70.0, 55.0, 35.0, 15.0):
            m_ref, r_ref, it_ref = hogbom(dirty, psf, 0.9, thr, 300)
            m, r, it = run(dirty, psf, torch.float64, 0.9, thr, 300)
            assert it == it_ref < 20
            assert np.array_equal(m, m_ref) and np.array_equal(r, r_ref)


def test_more_pixels_than_32_bits():
    """A peak past pixel 2^32 (FP32, 17 GB per image): its PSF is subtracted
    around it and nowhere else."""
    ny, nx = 65540, 65536
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    res = torch.zeros((ny, nx), dtype=torch.float32, device=DEV)
    psf, model = torch.zeros_like(res), torch.zeros_like(res)
    cy, cx = ny // 2, nx // 2
    psf[cy, cx] = 1.0
    psf[cy - 1, cx + 2] = 0.5
    y, x = 65537, 1234
    res[y, x] = 4.0
    assert lr.lr_hogbom(psf, res, model, 0.5, 0.0, 1) == 1
    want = {(y, x): 2.0, (y - 1, x + 2): -1.0}
    assert res.count_nonzero() == 2 and model.count_nonzero() == 1
    assert model[y, x] == 2.0
    for (i, j), v in want.items():
        assert res[i, j] == v
    del res, psf, model
    torch.cuda.empty_cache()
