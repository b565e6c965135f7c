"""bs_monopole_noalloc at the row limit n_tri nc = 2^31 - 1 (nc = 1): the rows' successors and the indices of
their k_perp exceed 32 bits.  All rows but a few lie above the k1 edges; those few, at both ends and where
3 t and the row cross 2^31 and 2^32, are binned."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, host, need_gpu, torch

pytestmark = pytest.mark.gpu

NT = 2 ** 31 - 1


def test_monopole_at_the_row_limit():
    need_gpu()
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB of device memory")
    rows = sorted({0, 1, 2 ** 31 // 3 - 1, 2 ** 31 // 3, 2 ** 31 // 3 + 1, 2 ** 32 // 3, 2 ** 32 // 3 + 1, NT - 8192,
                   NT - 8191, NT - 2, NT - 1})
    kperp = torch.full((NT, 3), 10.0, dtype=torch.float64, device="cuda")
    B = torch.full((NT, 1, 1), complex(1e30, 0.0), dtype=torch.complex128, device="cuda")
    for i, r in enumerate(rows):
        kperp[r] = torch.tensor([1.0, 0.9, 0.8], dtype=torch.float64)
        B[r] = float(2 ** i)
    edges = torch.tensor([0.5, 1.5, 2.0], dtype=torch.float64, device="cuda")
    mean = torch.empty((2, 5, 5), dtype=torch.float64, device="cuda")
    count = torch.empty((2, 5, 5), dtype=torch.int64, device="cuda")
    c = Ctx()
    try:
        bs.bs_monopole_noalloc(c.h, B, kperp, 1.0, edges, mean, count)
        n, m = host(count), host(mean)
        assert n.sum() == n.max() == len(rows)   # one shape: t = 0.9, mu = 0.65
        i = np.unravel_index(n.argmax(), n.shape)
        assert i == (0, 1, 4)
        assert m[i] == (2 ** len(rows) - 1) / len(rows)
    finally:
        c.close()
        del kperp, B
        torch.cuda.empty_cache()
