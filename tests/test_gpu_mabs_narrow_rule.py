"""The choice between 256 x 192 and narrow tiles of the split-BF16 contraction where the blocks do not fill the
chip: the chosen tiles are no slower than the 192-column ones (BS_MABS_M1 forces those)."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nc,rings,nu", [(64, 33, 4, 4), (64, 65, 4, 4), (64, 65, 4, 8), (64, 192, 4, 4), (128, 100, 3, 16)])
def test_no_slower_than_wide(monkeypatch, n, nc, rings, nu):
    need_gpu()
    c = Ctx()
    bs.bs_set_timing(c.h, True)
    h, nt = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, np.geomspace(1.0, (n - 1) // 3 + 0.5, rings + 1))
    V = torch.ones((nc, n, n // 2 + 1), dtype=torch.complex64, device="cuda")
    B = torch.empty((nt, nu, nc, nc), dtype=torch.float64, device="cuda")
    N = torch.empty((nt, nu, nc, nc), dtype=torch.int64, device="cuda")

    def us():
        t = []
        for _ in range(25):
            bs.bs_estimate_mabs(c.h, h, V, bs.BS_SPLIT_BF16, B, N, nu1=list(range(nu)))
            torch.cuda.synchronize()
            t.append(1e3 * bs.bs_last_timing(c.h)[1])
        return np.median(t[5:])

    try:
        monkeypatch.delenv("BS_MABS_M1", raising=False)
        rule = us()
        monkeypatch.setenv("BS_MABS_M1", str(min(16, nu)))
        wide = us()
        print(f"[narrow rule] n={n} nc={nc} nu1={nu}: {rule:.1f} us, wide {wide:.1f} us", flush=True)
        assert rule <= 1.06 * wide, (rule, wide)
    finally:
        bs.bs_free_bins(h)
        c.close()
