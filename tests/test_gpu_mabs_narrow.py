"""Split-BF16 MABS in narrow tiles: the same bits as in 256 x 192 tiles, at the edges of both.

Both kernels take, entry by entry, the same MFMAs in the same order with the same FP64 flushes, so B must be
equal bit for bit (BS_MABS_M1 forces the wide tiles).  Channels around the 16-row, 32-, 64- and 96-column
edges, first channels around units of 8 and in any order, pixel ranges of one and several flushes.  Parity
with the FP64 oracle is the other tests' (their few-channel cases take the narrow tiles).
"""
import numpy as np
import pytest

from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, torch
from test_gpu_mabs import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nc,nu1", [(16, 4, None), (16, 5, None), (32, 15, [14, 0, 3, 3, 9]), (32, 16, None),
                                      (32, 17, range(8)), (32, 31, range(9)), (32, 33, None), (32, 64, range(30)),
                                      (32, 65, range(7)), (32, 96, range(17)), (32, 97, range(4)),
                                      (32, 130, range(16)), (32, 200, range(5)), (192, 20, [19, 2, 4, 11])])
def test_narrow_tiles_give_the_same_bits(monkeypatch, n, nc, nu1):
    nu1 = None if nu1 is None else list(nu1)
    edges = np.geomspace(1.0, synth.default_umax(n) + 1.0, 4)
    V = synth.make_cube(synth.small_workload(n, nc), seed=nc)
    print(f"[narrow] n={n} nc={nc} nu1={nu1}", flush=True)
    c = Ctx()
    h, ncand = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, edges)
    got = []
    for m1 in (None, "4", "16"):
        if m1:
            monkeypatch.setenv("BS_MABS_M1", m1)
        else:
            monkeypatch.delenv("BS_MABS_M1", raising=False)
        B, N = run_gpu(c.h, h, V, bs.BS_SPLIT_BF16, ncand, len(nu1) if nu1 else nc, nc, nu1=nu1)
        got.append((B, N))
    bs.bs_free_bins(h)
    c.close()
    assert np.all(np.isfinite(got[0][0][got[0][1] > 0]))
    for B, N in got[1:]:
        assert np.array_equal(N, got[0][1])
        assert np.array_equal(B, got[0][0], equal_nan=True)
