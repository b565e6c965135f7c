"""Gridding at the edges of its layout: baseline counts around the block shares and the switch to the
large LDS region, counts that allow no 16-byte loads, channel groups of 1 to 9, grids smaller and larger than
the LDS region, baselines on the stored line q_v = 0 and off the grid, with and without flags, against the
oracle: counts bit for bit, sums within 1e-12 (FP64) of each cell's sum of |Re V| + |Im V|."""
import numpy as np
import pytest

from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, host, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("n,nco,avg,nvis", [(8, 1, 1, 3), (64, 2, 3, 2047), (66, 1, 4, 2050), (130, 3, 2, 8193), (256, 2, 5, 32767),
                                            (256, 1, 9, 32768), (200, 2, 4, 40002), (256, 5, 1, 65540), (32, 2, 4, 50000)])
@pytest.mark.parametrize("flagged", [False, True])
def test_layout_edges(ctx, n, nco, avg, nvis, flagged):
    du = synth.DU_G
    rng = np.random.default_rng(n * nvis)
    uv = synth.uv_tracks(nvis, nvis, 0.2 * du, 0.62 * n * du)
    k = nvis // 7
    uv[:k] = rng.uniform(-0.52 * n * du, 0.52 * n * du, (k, 2))     # far cells with few baselines
    uv[k:k + k // 2, 1] = rng.uniform(-0.4 * du, 0.4 * du, k // 2)  # the line q_v = 0, near and far
    nc = nco * avg
    vis = (rng.normal(size=(nc, nvis)) + 1j * rng.normal(size=(nc, nvis))).astype(np.complex64)
    flags = (rng.random((nc, nvis)) < 0.3).astype(np.uint8) if flagged else None
    if flagged:
        vis[flags != 0] = np.nan          # a flagged sample may hold anything
    print(f"[grid layout] n={n} nco={nco} avg={avg} nvis={nvis} flagged={flagged}", flush=True)
    Vg = torch.full((nco, n, n // 2 + 1), 3.0, dtype=torch.complex128, device="cuda")
    Ng = torch.full((nco, n, n // 2 + 1), 3, dtype=torch.int32, device="cuda")
    v64 = np.where(np.zeros_like(vis, dtype=bool) if flags is None else flags != 0, 0, vis).astype(np.complex128)
    rV, rN = oe.grid_visibilities(uv, v64, flags, n, du, avg)
    mag, _ = oe.grid_visibilities(uv, np.abs(v64.real) + np.abs(v64.imag), flags, n, du, avg)
    for _ in range(2):   # the second call reuses the workspaces
        bs.bs_grid_visibilities(ctx, n, du, cuda(uv), cuda(vis), Vg, Ng, flags=None if flags is None else cuda(flags),
                                chan_avg=avg, precision=bs.BS_FP64)
        assert np.array_equal(host(Ng), rN)
        assert np.all(np.abs(host(Vg) - rV) <= 1e-12 * np.abs(mag) + 1e-300)
