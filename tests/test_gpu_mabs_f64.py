"""The FP64 contraction at the edges of its tiles (16 nu2 rows and 1-4 column tiles of 16 a wave, waves
spread 4 x 1, 2 x 2 or 1 x 4 over (nu1, nu2)) and of its 16-pixel stages, as data kernel (unit
weights) and as count kernel (per-cell N_g), against the oracle: counts bit for bit, B within the
FP64 bar of 1e-10 relative (sums of at most 1296 products in float64)."""
import numpy as np
import pytest

from oracle import bins as ob
from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, compare_B, cuda, host, torch, vis_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


# n = 18: 324 pixels, not a multiple of the 16-pixel stage; n = 36: 1296 pixels
@pytest.mark.parametrize("n,nc,n_nu1", [(18, 5, 5), (18, 16, 1), (18, 17, 2), (36, 33, 3), (18, 48, 5), (18, 65, 8),
                                        (18, 96, 9), (36, 16, 16)])
@pytest.mark.parametrize("counts", [False, True])
def test_tile_edges(ctx, n, nc, n_nu1, counts):
    edges = np.geomspace(1.0, (n - 1) // 3 + 1.0, 4)
    V = synth.make_cube(synth.small_workload(n, nc), seed=n + nc)
    nu1 = [(7 * i) % nc for i in range(n_nu1)] if n_nu1 < nc else list(range(nc))
    wt, kw = None, {}
    if counts:
        ng = np.random.default_rng(nc).integers(0, 4, size=(nc, n, n // 2 + 1)).astype(np.uint16)
        neg = (-np.arange(n)) % n
        ng[:, :, 0] = np.maximum(ng[:, :, 0], ng[:, neg, 0])
        wt, kw = oe.Weights(ng=ng), {"ng": cuda(ng.view(np.int16))}
    b = ob.make_bins(ob.RING_U, n, nc, edges)
    f = oe.MabsFields(b, V, wt)
    Bref, Nref, S, _ = oe.estimate_mabs(b, V, wt, nu1=nu1, fields=f)
    A = np.stack([oe.triple_sum(np.abs(f.data(x).reshape(nc, -1))[nu1], np.abs(f.data(y).reshape(nc, -1)),
                                np.abs(f.data(z).reshape(nc, -1))) for x, y, z in b.triangles])
    scale = np.where(Nref > 0, n * n * A / np.maximum(Nref, 1), 0.0)
    print(f"[mabs f64] n={n} nc={nc} n_nu1={n_nu1} counts={counts}", flush=True)
    h, nt = bs.bs_make_bins(ctx, bs.BS_RING_U, n, nc, edges)
    try:
        B = torch.empty((nt, len(nu1), nc, nc), dtype=torch.float64, device="cuda")
        N = torch.empty((nt, len(nu1), nc, nc), dtype=torch.int64, device="cuda")
        bs.bs_estimate_mabs(ctx, h, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, B, N, nu1=nu1, **kw)
        Bg, Ng = host(B), host(N)
    finally:
        bs.bs_free_bins(h)
    assert np.array_equal(Ng, Nref)
    compare_B(Bg, Bref, Nref, scale, 1e-10)
