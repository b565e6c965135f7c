"""Calls in a row on one context give what a fresh context gives, bit for bit: weights whose contents
change in place, masks, unweighted calls, precisions and streams between them (the context reuses the
prepared 3D estimate and tables that did not change)."""
import numpy as np
import pytest

from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, host, need_gpu, torch, vis_tensor

pytestmark = pytest.mark.gpu

N, NC = 16, 32
EDGES = 2 * np.pi * np.geomspace(1.0 / N, 5.5 / N, 6)


def est3d(ctx, bins, V, prec, ncand, **kw):
    B = torch.empty(ncand, dtype=torch.float64, device="cuda")
    T = torch.empty(ncand, dtype=torch.int64, device="cuda")
    E = torch.empty(ncand, dtype=torch.float64, device="cuda")
    bs.bs_estimate_3d(ctx, bins, vis_tensor(V, prec), prec, B, T, E, **kw)
    return host(B), host(T), host(E)


def bins3(ctx):
    return bs.bs_make_bins(ctx, bs.BS_SHELL_K, N, NC, EDGES, du_lambda=1.0, r_mpc=float(N), rprime_mpc_per_mhz=1.0,
                           dnu_mhz=float(N) / NC)


def same(a, b):
    return all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b))


@pytest.mark.parametrize("prec", [bs.BS_FP64, bs.BS_FP32, bs.BS_SPLIT_BF16])
def test_3d_weights_change_in_place(prec):
    need_gpu()
    V = synth.make_cube(synth.small_workload(N, NC), seed=4)
    rng = np.random.default_rng(1)
    cw, um = cuda(np.ones(NC), np.float32), cuda(synth.disk_mask(N))
    steps = []
    for k in range(7):
        w = (rng.random(NC) > 0.2 * k).astype(np.float32) if k != 5 else rng.random(NC).astype(np.float32)
        m = synth.disk_mask(N, 5.0 - (k % 3))
        steps.append((w, m, k))
    c = Ctx()
    h, n = bins3(c.h)
    try:
        for w, m, k in steps:
            cw.copy_(torch.from_numpy(w))
            um.copy_(torch.from_numpy(m))
            kw = [{}, {"chan_w": cw}, {"uv_mask": um}, {"chan_w": cw, "uv_mask": um}][k % 4]
            got = est3d(c.h, h, V, prec, n, **kw)
            f = Ctx()
            hf, _ = bins3(f.h)
            ref = est3d(f.h, hf, V, prec, n, **kw)
            bs.bs_free_bins(hf)
            f.close()
            assert same(got, ref), k
            if "chan_w" in kw:
                rho3 = oe.rho3(oe.Weights(chan_w=w.astype(np.float64)), NC)
                assert np.allclose(got[2], got[1] * rho3, rtol=1e-14)
    finally:
        bs.bs_free_bins(h)
        c.close()


def test_tables_follow_selection_and_stream():
    need_gpu()
    n, nc = 16, 6
    edges = np.geomspace(1.0, 6.0, 5)
    V = synth.make_cube(synth.small_workload(n, nc), seed=2)
    c = Ctx()
    h, nt = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, edges)
    tri = bs.bs_bins_triangles(h, nt, 4)[0]
    s2 = torch.cuda.Stream()

    def call(ctx, bins, sel, nu1):
        B = torch.empty((len(sel), len(nu1), nc, nc), dtype=torch.float64, device="cuda")
        T = torch.empty((len(sel), len(nu1), nc, nc), dtype=torch.int64, device="cuda")
        bs.bs_estimate_mabs(ctx, bins, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, B, T, tri3=sel, nu1=nu1)
        return host(B), host(T)

    try:
        for k, (sel, nu1) in enumerate([(tri, [0, 1]), (tri[::-1], [0, 1]), (tri[::-1], [3, 2]), (tri[:2], [5]), (tri, [0, 1])]):
            if k == 4:
                torch.cuda.synchronize()
                bs.bs_set_stream(c.h, s2.cuda_stream)
            got = call(c.h, h, sel, nu1)
            f = Ctx()
            hf, _ = bs.bs_make_bins(f.h, bs.BS_RING_U, n, nc, edges)
            ref = call(f.h, hf, sel, nu1)
            bs.bs_free_bins(hf)
            f.close()
            assert same(got, ref), k
    finally:
        bs.bs_free_bins(h)
        c.close()
