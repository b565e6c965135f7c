"""The ergodic collapse where its waves meet the ends of the band (rows of 2 nc - 1 separations shorter
and longer than a wave, circular wrap-around), with per-cell counts that differ by channel and with
flagged channels, against the oracle's collapse of the full MABS: counts bit for bit, means of at most
nc FP64 estimates within 1e-10 of the mean absolute estimate."""
import numpy as np
import pytest

from oracle import bins as ob
from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, host, torch, vis_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("nc", [2, 7, 33, 40])
@pytest.mark.parametrize("collapse", [1, 2])
@pytest.mark.parametrize("counts", [False, True])
def test_collapse_edges(ctx, nc, collapse, counts):
    n = 16
    edges = np.array([1.0, 2.2, 4.0])
    V = synth.make_cube(synth.small_workload(n, nc), seed=nc)
    rng = np.random.default_rng(nc)
    if counts:
        ng = rng.integers(0, 3, size=(nc, n, n // 2 + 1)).astype(np.uint16)
        neg = (-np.arange(n)) % n
        ng[:, :, 0] = np.maximum(ng[:, :, 0], ng[:, neg, 0])
        wt, kw = oe.Weights(ng=ng), {"ng": cuda(ng.view(np.int16))}
    else:
        cw = (rng.random(nc) > 0.2).astype(np.float64)
        cw[0] = 1.0
        wt, kw = oe.Weights(chan_w=cw), {"chan_w": cuda(cw, np.float32)}
    b = ob.make_bins(ob.RING_U, n, nc, edges)
    B, N, _, _ = oe.estimate_mabs(b, V, wt, fields=oe.MabsFields(b, V, wt))
    Bref, Nnu, Ntot = oe.collapse_mabs(B, N, circular=collapse == 2)
    mag, _, _ = oe.collapse_mabs(np.abs(np.nan_to_num(B)), N, circular=collapse == 2)
    print(f"[collapse] nc={nc} collapse={collapse} counts={counts}", flush=True)
    h, nt = bs.bs_make_bins(ctx, bs.BS_RING_U, n, nc, edges)
    try:
        shp = Bref.shape
        Bg = torch.empty(shp, dtype=torch.float64, device="cuda")
        Ng = torch.empty(shp, dtype=torch.int64, device="cuda")
        Nn = torch.empty(shp, dtype=torch.int32, device="cuda")
        bs.bs_estimate_mabs(ctx, h, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, Bg, Ng, Nn, collapse=collapse, **kw)
        Bg, Ng, Nn = host(Bg), host(Ng), host(Nn)
    finally:
        bs.bs_free_bins(h)
    assert np.array_equal(Nn, Nnu) and np.array_equal(Ng, Ntot)
    ok = Nnu > 0
    assert np.all(np.isnan(Bg[~ok]))
    assert np.all(np.abs(Bg[ok] - Bref[ok]) <= 1e-10 * mag[ok])
