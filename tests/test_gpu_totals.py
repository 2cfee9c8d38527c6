"""GPU: sums of weights and class counts of a gridding call, which each
workgroup of the presum totals before it adds them: planes that change
within a wavefront, within a workgroup and between workgroups, skipped
channels, flags, dropped samples, rows with and without a period."""

import numpy as np
import pytest

import oracle
import synth
from oracle.cfbuild import TERM_PS
from oracle.native import Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_17187_amd import lr  # noqa: E402
from paper_2508_17187_amd import workload as W  # noqa: E402

# output plane of each channel (-1: skipped)
PLANES = {"one": [0], "alternate": [0, 1, 2] * 3, "blocks": [0] * 8 + [1] * 8 + [-1] * 8 + [2] * 9,
          "skipped": [-1, -1]}


@pytest.mark.parametrize("npol", [1, 2, 4])
@pytest.mark.parametrize("planes", list(PLANES))
@pytest.mark.parametrize("shuffled", [False, True])
def test_totals_match_the_oracle(npol, planes, shuffled):
    cp = PLANES[planes]
    wl = synth.tiny_workload(n_ant=7, n_time=70, nchan=len(cp), npol=npol, nx=64, ny=48,
                             cell_arcsec=9.0, diameter_m=4000.0, oversample=8, terms=TERM_PS,
                             nplane=3, chan_plane=cp, cfg_id=260)
    rng = np.random.default_rng(260)
    wl.weight[:] = rng.random(wl.weight.shape) + 0.5
    wl.weight[rng.random(wl.weight.shape) < 0.1] = 0.0
    if shuffled:
        i = rng.permutation(wl.obs.nrow)
        wl.obs.uvw, wl.vis, wl.weight = wl.obs.uvw[i], wl.vis[i], wl.weight[i]
    cf = W.build_cf(wl, lr.LR_F64)
    v = W.device_vis(wl, lr.LR_F64)
    ref_s, ref_c = Problem.from_workload(wl, oracle.build_cf(wl.grid, wl.cf)).sumwt(wl.weight)
    for call in ("grid", "sumwt"):
        s = torch.ones((3, npol), dtype=torch.float64, device="cuda")
        c = torch.ones(3, dtype=torch.int64, device="cuda")
        if call == "grid":
            lr.lr_grid(cf, v, lr.LR_F64, W.empty_grid(wl, lr.LR_F64), s, c)
        else:
            lr.lr_sumwt(cf, v, lr.LR_F64, s, c)
        assert np.array_equal(c.cpu().numpy() - 1, ref_c)
        # a sum of at most 1e5 weights of about 1 in any order: 1e5 roundings of
        # 1e5 * 2^-53 at most, 1e-16 relative each
        assert np.abs(s.cpu().numpy() - 1 - ref_s).max() <= 1e-11 * max(np.abs(ref_s).max(), 1.0)
