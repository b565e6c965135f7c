"""A moment's weight carries its norm before it meets the value: with one non-zero cell a bin (nc = 2, a triangle a
k1 bin) the l <= 1 moments are, bit for bit, (norm Q cos) v over the bin's count as plain IEEE operations give it."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, cuda, host, need_gpu, torch

pytestmark = pytest.mark.gpu


def test_single_cells():
    need_gpu()
    nt, unit = 64, 0.02
    rng = np.random.default_rng(5)
    kp = np.geomspace(1.0, 40.0, nt)[:, None] * np.stack([np.ones(nt), rng.uniform(0.6, 0.95, nt), rng.uniform(0.4, 0.58, nt)], 1)
    v = rng.standard_normal(nt)
    B = np.zeros((nt, 2, 2), dtype=np.complex128)
    B[:, 1, 1] = v                                     # k_par1 = k_par2 = -unit, k_par3 = 2 unit
    edges = np.concatenate([[0.5], 0.5 * (kp[1:, 0] + kp[:-1, 0]), [80.0]])
    k = np.array([0.0, -unit])
    cnt = np.zeros((nt, 5, 5), dtype=np.int64)
    want = np.zeros((3, nt, 5, 5))
    for t in range(nt):
        for a in range(2):
            for b in range(2):
                par = np.array([k[a], k[b], -(k[a] + k[b])])
                s = kp[t] * kp[t] + par * par
                o = np.argsort(-s, kind="stable")
                hi, mid, lo = s[o]
                k1, k2 = np.sqrt(hi), np.sqrt(mid)
                mu = np.clip(((hi + mid) - lo) / (2.0 * (k1 * k2)), 0.5, 1.0)
                tt = np.clip(k2 / k1, 0.5, 1.0)
                j = np.searchsorted(edges, k1, side="right") - 1
                i = (j, sum(mu >= x for x in (0.6, 0.7, 0.8, 0.9)), sum(tt >= x for x in (0.6, 0.7, 0.8, 0.9)))
                cnt[i] += 1
                if (a, b) == (1, 1):
                    pz = par[o[0]] / k1
                    px = (par[o[1]] / k2 + mu * pz) / np.sqrt(1.0 - mu * mu)
                    assert px * px < 1.0 - pz * pz
                    assert want[0][i] == 0.0           # a bin of its own
                    want[0][i] = v[t]
                    want[1][i] = (3.0 * pz) * v[t]
                    want[2][i] = (((3.0 * np.sqrt(0.5)) * -1.0) * px) * v[t]
    with np.errstate(invalid="ignore"):
        want = np.where(cnt > 0, want / cnt, np.nan)
    M = torch.empty((3, nt, 5, 5), dtype=torch.float64, device="cuda")
    N = torch.empty((nt, 5, 5), dtype=torch.int64, device="cuda")
    c = Ctx()
    try:
        bs.bs_multipoles(c.h, cuda(B), kp, unit, edges, 1, M, N)
        assert np.array_equal(host(N), cnt)
        for i in range(3):
            assert np.array_equal(host(M)[i], want[i], equal_nan=True), i
    finally:
        c.close()
