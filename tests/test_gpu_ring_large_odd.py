"""Ring fields of the grids whose columns did not fit a block's LDS at any fold (n = 2^a 3^b with few factors of
two: 324, 486, 648, 864, 972): data and count fields and FP64 MABS counts against the oracle.

Tolerance: FP64 2e-12 and FP32 5e-6 of max |F| (transforms of up to 972 points, see test_gpu_ring_fields)."""
import numpy as np
import pytest

from oracle import bins as ob
from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, host, need_gpu, torch, vis_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [324, 486, 648, 864, 972])
@pytest.mark.parametrize("precision", [bs.BS_FP64, bs.BS_FP32])
def test_ring_fields(n, precision):
    need_gpu()
    top = (n - 1) // 3
    edges = np.array([1.0, 2.3, 0.4 * top, top + 1.0])
    V = synth.make_cube(synth.small_workload(n, 2), seed=n)
    b = ob.make_bins(ob.RING_U, n, 2, edges)
    f = oe.MabsFields(b, V)
    print(f"[ring large odd] n={n} precision={precision}", flush=True)
    c = Ctx()
    h, nt = bs.bs_make_bins(c.h, bs.BS_RING_U, n, 2, edges)
    try:
        F = torch.empty((3, 2, n, n), dtype=torch.float64 if precision == bs.BS_FP64 else torch.float32, device="cuda")
        I = torch.empty((3, 2, n, n), dtype=torch.float64, device="cuda")
        bs.bs_filter_fields(c.h, h, vis_tensor(V, precision), 0, precision, F, I)
        B = torch.empty((nt, 2, 2, 2), dtype=torch.float64, device="cuda")
        N = torch.empty((nt, 2, 2, 2), dtype=torch.int64, device="cuda")
        bs.bs_estimate_mabs(c.h, h, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, B, N)
        Fg, Ig, Ng, tri = host(F).astype(np.float64), host(I), host(N), bs.bs_bins_triangles(h, nt, 3)[0]
    finally:
        bs.bs_free_bins(h)
        c.close()
    tol = 2e-12 if precision == bs.BS_FP64 else 5e-6
    cnt = []
    for j in range(3):
        Fr, Ir = f.data(j).reshape(2, n, n), f.count(j).reshape(-1, n, n)
        cnt.append(Ir[0])
        assert np.max(np.abs(Fg[j] - Fr)) <= tol * np.max(np.abs(Fr)), j
        assert np.max(np.abs(Ig[j] - Ir)) <= 2e-12 * np.max(np.abs(Ir)), j
    for t, (i, j, k) in enumerate(tri):
        want = float(n) ** 4 * float(np.sum((cnt[i] * cnt[j] * cnt[k]).astype(np.longdouble)))
        assert abs(want - round(want)) < 0.25 and np.all(Ng[t] == round(want)), (t, want)
