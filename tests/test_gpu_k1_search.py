"""The k1 bin search at every first step it can start from and at the switch between the two kernels (14 and
15 bins): nc = 1, so that a triangle is one cell and k1 its largest k_perp, on the edges, one rounding to either
side of them, between and outside them.  Counts equal numpy's search, sums the exact small integers."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, cuda, host, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk", [1, 2, 3, 6, 7, 13, 14, 15, 16, 30, 31, 62, 63, 64])
def test_edges(nk):
    need_gpu()
    e = np.geomspace(0.07, 3.1, nk + 1)
    k1 = np.concatenate([e, np.nextafter(e, 0), np.nextafter(e, 9), np.sqrt(e[1:] * e[:-1]), [0.01, 0.069, 3.2, 40.0]])
    # k1 as the kernel forms it: the square root of the squared side
    k1 = np.sqrt(k1 * k1)
    nt = k1.size
    kp = np.stack([0.95 * k1, k1, 0.9 * k1], 1)
    val = np.arange(1.0, nt + 1)
    want_n = np.zeros((nk, 5, 5), dtype=np.int64)
    want_s = np.zeros((nk, 5, 5))
    j = np.searchsorted(e, k1, side="right") - 1
    for t in np.nonzero((j >= 0) & (j < nk))[0]:
        q = np.sort(kp[t] * kp[t])
        a, b = np.sqrt(q[2]), np.sqrt(q[1])
        mu, tt = ((q[2] + q[1]) - q[0]) / (2.0 * (a * b)), b / a
        i = (j[t], sum(mu >= x for x in (0.6, 0.7, 0.8, 0.9)), sum(tt >= x for x in (0.6, 0.7, 0.8, 0.9)))
        want_n[i] += 1
        want_s[i] += val[t]
    B = cuda(val.astype(np.complex128).reshape(nt, 1, 1))
    with np.errstate(invalid="ignore"):
        want = want_s / want_n
    c = Ctx()
    try:
        for call in ("host", "noalloc", "multi"):
            N = torch.empty((nk, 5, 5), dtype=torch.int64, device="cuda")
            M = torch.empty((nk, 5, 5), dtype=torch.float64, device="cuda")
            if call == "host":
                bs.bs_monopole(c.h, B, kp, 1.0, e, M, N)
            elif call == "noalloc":
                bs.bs_monopole_noalloc(c.h, B, cuda(kp), 1.0, cuda(e), M, N)
            else:
                bs.bs_multipoles(c.h, B, kp, 1.0, e, 0, M.view(1, nk, 5, 5), N)
            assert np.array_equal(host(N), want_n), call
            assert np.array_equal(host(M), want, equal_nan=True), call
    finally:
        c.close()
