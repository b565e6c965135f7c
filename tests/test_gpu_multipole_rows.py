"""Multipole moments and monopole where rows, batches and merged lanes run out unevenly.

Many triangles of a narrow band (a wave has more than 64 rows), few triangles of a wide one (rows with more
cells than a batch), one bin for every cell (all lanes merge) and edges that split neighbours (64 k1 bins go
with l <= 1: the entry point takes 6400 values at most).  Counts bit
for bit, moments within 1e-11 (2l + 1) of the bin's mean |Re B| (FP64 sums in another order, as for the
other sizes); an infinite value makes its bin's moments what the sum of its weighted terms is.
"""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, cuda, host, torch
from oracle import estimator as oe
from test_gpu_multipoles import check, random_triangles, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,nt,nk,lmax", [(4, 70000, 3, 1), (5, 1, 1, 4), (700, 1, 1, 4), (700, 2, 9, 4),
                                           (64, 40, 17, 4), (257, 3, 64, 1)])
def test_rows(nc, nt, nk, lmax):
    rng = np.random.default_rng(nc + nt)
    kperp = random_triangles(rng, nt, 0.05)
    unit = 0.02 if nc < 100 else 0.001
    B = rng.normal(size=(nt, nc, nc)) + 1j * rng.normal(size=(nt, nc, nc))
    edges = np.geomspace(0.01, 0.3 + unit * nc, nk + 1)
    print(f"[multi rows] nc={nc} nt={nt} nk={nk}", flush=True)
    c = Ctx()
    got = run(c.h, cuda(B), kperp, unit, edges, lmax)
    mean = torch.empty((nk, 5, 5), dtype=torch.float64, device="cuda")
    cnt = torch.empty((nk, 5, 5), dtype=torch.int64, device="cuda")
    bs.bs_monopole(c.h, cuda(B), kperp, unit, edges, mean, cnt)
    mean, cnt = host(mean), host(cnt)
    c.close()
    check(got, B, kperp, unit, edges, lmax, f"nc={nc} nt={nt}")
    rm, rc = oe.bs_monopole(B, kperp, unit, edges)
    mag, _ = oe.bs_monopole(np.abs(B.real), kperp, unit, edges)
    ok = rc > 0
    assert np.array_equal(cnt, rc) and np.all(np.isnan(mean[~ok]))
    assert np.all(np.abs(mean[ok] - rm[ok]) <= 1e-11 * mag[ok] + 1e-300)


def test_an_infinite_value():
    nc = 24
    rng = np.random.default_rng(3)
    kperp = random_triangles(rng, 1, 0.05)
    B = rng.normal(size=(1, nc, nc)) + 0j
    edges = np.geomspace(0.01, 1.0, 4)
    c = Ctx()
    ref, rc = run(c.h, cuda(B), kperp, 0.02, edges, 4)
    B[0, 3, 5] = np.inf
    one = np.zeros_like(B)
    one[0, 3, 5] = 1.0   # the weights of that cell over its bin's count
    w, _ = run(c.h, cuda(one), kperp, 0.02, edges, 4)
    got, cnt = run(c.h, cuda(B), kperp, 0.02, edges, 4)
    c.close()
    assert np.array_equal(cnt, rc)
    hit = np.nan_to_num(w) != 0.0
    assert hit.any()
    assert np.array_equal(got[hit], np.copysign(np.inf, w[hit]))
    other = ~hit.any(axis=0) & (rc > 0)
    assert np.allclose(got[:, other], ref[:, other], rtol=0, atol=1e-11)
