"""Counts from per-channel fields are certified by the pixel chunks they are summed in: a call whose tiles
alone fill the chip still splits its pixels where one chunk is too long to certify, at 64 entries a
triangle (a block an entry) and beyond (MFMA tiles).  Exact counts: those of a uv mask of ones."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, host, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [bs.BS_FP64, bs.BS_SPLIT_BF16])
@pytest.mark.parametrize("nc, n_nu1", [(4, 4), (12, 12)])
def test_many_triangles_on_a_large_grid(nc, n_nu1, prec):
    need_gpu()
    n = 768
    edges = np.concatenate([np.arange(1.0, 9.0), [255.5]])   # eight narrow rings and one of 200,000 cells
    c = Ctx()
    h, nt = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, edges)
    rdt = torch.float64 if prec == bs.BS_FP64 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(3)
    V = torch.view_as_complex(torch.randn(nc, n, n // 2 + 1, 2, generator=g, device="cuda", dtype=rdt))
    shape = (nt, n_nu1, nc, nc)
    try:
        got = []
        for kw in ({}, {"ng": torch.ones((nc, n, n // 2 + 1), dtype=torch.int16, device="cuda")}):
            B = torch.empty(shape, dtype=torch.float64, device="cuda")
            T = torch.empty(shape, dtype=torch.int64, device="cuda")
            bs.bs_estimate_mabs(c.h, h, V, prec, B, T, nu1=list(range(n_nu1)), **kw)
            got.append((host(B), host(T)))
        assert bs.bs_last_count_dev(c.h) <= bs.bs_last_count_bound(c.h) < 0.5
        (B0, T0), (B1, T1) = got
        assert np.array_equal(T0, T1) and T0.max() > 1e9
        ok = T0 > 0
        assert np.array_equal(np.isnan(B1), ~ok)
        # equal fields; the partial sums are split differently, n^2 terms whose largest share is B_abs
        tol = 1e-10 if prec == bs.BS_FP64 else 1e-4
        assert np.abs(B1 - B0)[ok].max() <= tol * np.sqrt(np.mean(B0[ok] ** 2))
    finally:
        bs.bs_free_bins(h)
        c.close()
