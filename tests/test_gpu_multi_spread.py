"""The rows that hold cells are spread over the blocks in small calls: a call in which a fifth of the rows are
binned takes no longer than one in which all of them are."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, need_gpu, torch

pytestmark = pytest.mark.gpu


def test_few_rows_with_cells():
    need_gpu()
    nc, nt, nk, lmax = 24, 4, 12, 4
    rng = np.random.default_rng(nc)
    kp = np.sort(rng.uniform(0.05, 0.6, (nt, 3)), axis=1)[:, ::-1].copy()
    X = torch.ones((nt, nc, nc), dtype=torch.complex128, device="cuda")
    C = torch.empty((nk, 5, 5), dtype=torch.int64, device="cuda")
    M = torch.empty((15, nk, 5, 5), dtype=torch.float64, device="cuda")
    c = Ctx()
    bs.bs_set_timing(c.h, True)

    def kernel_us(kmax):
        t = []
        for _ in range(60):
            bs.bs_multipoles(c.h, X, kp, 2 * np.pi / (0.75 * nc), np.geomspace(0.05, kmax, nk + 1), lmax, M, C)
            t.append(1e3 * bs.bs_last_timing(c.h)[1])
        return np.median(t[10:])

    try:
        few, every = kernel_us(0.8), kernel_us(8.0)
        print(f"[multi spread] few rows {few:.1f} us, all rows {every:.1f} us", flush=True)
        assert few <= 1.1 * every, (few, every)
    finally:
        c.close()
