"""Gridding with staged far baselines: every one staged, and more of them than the staging space holds.

All channels hold the same visibilities, so each channel's cells must match the oracle's for one: counts
bit for bit, sums within 1e-12 (FP64 sums in another order) of each cell's sum of |Re V| + |Im V|.  The
outputs of cells that nothing reaches must be zero.
"""
import numpy as np
import pytest

from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, host, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nco,nvis", [(256, 1000, 60000), (256, 1000, 50000), (140, 7, 33333), (128, 9, 40000), (4, 3, 40000)])
def test_staging(n, nco, nvis):
    du = synth.DU_G
    rng = np.random.default_rng(n + nvis)
    uv = rng.uniform(-0.51 * n * du, 0.51 * n * du, (nvis, 2))   # nearly all of them far
    uv[:200, 1] = rng.uniform(-0.4 * du, 0.4 * du, 200)          # the line q_v = 0
    vis = (rng.normal(size=(1, nvis)) + 1j * rng.normal(size=(1, nvis))).astype(np.complex64)
    print(f"[grid staging] n={n} nco={nco} nvis={nvis}", flush=True)
    v64 = vis.astype(np.complex128)
    rV, rN = oe.grid_visibilities(uv, v64, None, n, du, 1)
    mag, _ = oe.grid_visibilities(uv, np.abs(v64.real) + np.abs(v64.imag), None, n, du, 1)
    c = Ctx()
    vd = cuda(vis).repeat(nco, 1)
    Vg = torch.full((nco, n, n // 2 + 1), 3.0, dtype=torch.complex128, device="cuda")
    Ng = torch.full((nco, n, n // 2 + 1), 3, dtype=torch.int32, device="cuda")
    bound = cuda(1e-12 * np.abs(mag) + 1e-300)
    for _ in range(2):   # the second call reuses the workspaces
        bs.bs_grid_visibilities(c.h, n, du, cuda(uv), vd, Vg, Ng, chan_avg=1, precision=bs.BS_FP64)
        assert torch.equal(Ng, cuda(rN).to(torch.int32).expand_as(Ng))
        assert bool(((Vg - cuda(rV)).abs() <= bound).all())
        Vg.fill_(5.0)
    c.close()
