"""Ring fields where their two passes have edges: rows whose column values fill the whole row (support
radius n / 2 - 1), rings without a cell, one column only, lengths with factors of three, folded FP32
columns (n = 256), flags, per-cell counts and count fields, against the oracle's fields.

Tolerance: FP64 1e-12 and FP32 3e-6 of max |F| (two transforms of at most 256 points; a rounding error
of about eps log2 n per transform)."""
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


@pytest.mark.parametrize("n,nc,umax", [(8, 3, 3.0), (16, 2, 0.0), (18, 3, 8.0), (48, 1, 0.0), (54, 2, 26.0), (64, 3, 31.0), (96, 1, 40.0), (128, 1, 0.0), (192, 1, 0.0),
                                       (256, 2, 0.0), (256, 1, 127.0)])
@pytest.mark.parametrize("precision", [bs.BS_FP64, bs.BS_FP32])
@pytest.mark.parametrize("weights", ["unit", "flags", "counts"])
def test_ring_fields(ctx, n, nc, umax, precision, weights):
    top = umax if umax > 0 else (n - 1) // 3
    # the first ring holds one column's reach, the second has no cell (between 1 and sqrt 2), the last may be empty
    edges = np.array([1.0, 1.1, 1.4, 2.3, 0.6 * top + 1.2, top + 1.0, top + 2.0])
    V = synth.make_cube(synth.small_workload(n, nc), seed=n + nc)
    wt, kw = None, {}
    if weights == "flags":
        cw, um = (np.arange(nc) % 2 == 0).astype(np.float64), synth.disk_mask(n, 0.8 * top)
        wt, kw = oe.Weights(uv_mask=um, chan_w=cw), {"uv_mask": cuda(um), "chan_w": cuda(cw, np.float32)}
    elif weights == "counts":
        ng = np.random.default_rng(n).integers(0, 4, size=(nc, n, n // 2 + 1)).astype(np.uint16)
        neg = (-np.arange(n)) % n
        ng[:, :, 0] = np.maximum(ng[:, :, 0], ng[:, neg, 0])
        wt, kw = oe.Weights(ng=ng), {"ng": cuda(ng.view(np.int16))}
    b = ob.make_bins(ob.RING_U, n, nc, edges, umax=umax if umax > 0 else None)
    f = oe.MabsFields(b, V, wt)
    print(f"[ring fields] n={n} nc={nc} umax={umax} precision={precision} {weights}", flush=True)
    h, _ = bs.bs_make_bins(ctx, bs.BS_RING_U, n, nc, edges, umax=umax)
    try:
        F = torch.full((6, nc, n, n), 7.0, dtype=torch.float64 if precision == bs.BS_FP64 else torch.float32, device="cuda")
        I = torch.full((6, nc, n, n), 7.0, dtype=torch.float64, device="cuda")
        bs.bs_filter_fields(ctx, h, vis_tensor(V, precision), 0, precision, F, I, **kw)
        Fg, Ig = host(F).astype(np.float64), host(I)
    finally:
        bs.bs_free_bins(h)
    tol = 1e-12 if precision == bs.BS_FP64 else 3e-6
    for j in range(6):
        Fr, Ir = f.data(j).reshape(nc, n, n), np.broadcast_to(f.count(j).reshape(-1, n, n), (nc, n, n))
        assert np.max(np.abs(Fg[j] - Fr)) <= tol * max(np.max(np.abs(Fr)), 1e-300), j
        assert np.max(np.abs(Ig[j] - Ir)) <= 1e-12 * max(np.max(np.abs(Ir)), 1e-300), j
