"""The FP64 3D contraction from one pair tile to as many as the shells need, with third fields past 15,
voxel counts that are no multiple of its 128-voxel slabs and single-block cubes (26 such shells need more
than the 112 pairs the library takes): counts bit for bit
against the oracle's exact counts, B within 1e-10 relative (or of B_abs where the sum cancels)."""
import numpy as np
import pytest

from oracle import bins as ob
from oracle import counts as oc
from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, compare_B, host, torch, vis_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("n,nc,shells", [(8, 2, 1), (12, 6, 2), (16, 18, 4), (18, 16, 8), (16, 32, 12), (24, 24, 16),
                                         (24, 24, 20)])
def test_counts_and_fp64_estimate(ctx, n, nc, shells):
    top = (n - 1) // 3 + 0.5
    edges = 2 * np.pi / n * np.linspace(0.9, top, shells + 1)
    kw = dict(du=1.0, r_mpc=float(n), rprime=1.0, dnu=float(n) / nc)
    V = synth.make_cube(synth.small_workload(n, nc), seed=n + shells)
    b = ob.make_bins(ob.SHELL_K, n, nc, edges, **kw)
    T, _ = oc.exact_counts(b)
    f = oe.ShellFields(b, V)
    Bref, T3, neff, _, _ = oe.estimate_3d(b, V, fields=f, counts=T)
    A = np.array([np.sum(np.abs(f.data(i) * f.data(j) * f.data(k))) for i, j, k in b.triangles])
    scale = np.where(T > 0, nc * n * n * A / np.maximum(neff, 1.0), 0.0)
    print(f"[contract64] n={n} nc={nc} shells={shells} triangles={len(b.triangles)}", flush=True)
    h, nt = bs.bs_make_bins(ctx, bs.BS_SHELL_K, n, nc, edges, du_lambda=1.0, r_mpc=float(n), rprime_mpc_per_mhz=1.0,
                            dnu_mhz=float(n) / nc)
    try:
        B = torch.empty(nt, dtype=torch.float64, device="cuda")
        N = torch.empty(nt, dtype=torch.int64, device="cuda")
        bs.bs_estimate_3d(ctx, h, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, B, N)
        Bg, Ng = host(B), host(N)
    finally:
        bs.bs_free_bins(h)
    assert nt == len(b.triangles) and np.array_equal(Ng, T)
    compare_B(Bg, Bref, T, scale, 1e-10)
