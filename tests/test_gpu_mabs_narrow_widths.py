"""Every width of the narrow split-BF16 tiles (BS_MABS_NJ) against the 256 x 192 tiles, bit for bit, whatever the
rule would take: channels around the 16-row and 32-, 64- and 96-column edges, first channels around units of 8 and
in any order, an odd number of 32-pixel stages, and pixel chunks of two and of four and a half FP64 flushes
(BS_MABS_KCHUNKS=1: 16384 and 36864 pixels, a flush every 8192)."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, need_gpu
from test_gpu_mabs import run_gpu

pytestmark = pytest.mark.gpu

CASES = [(16, 4, None, None), (32, 15, [14, 0, 3, 3, 9], None), (32, 16, None, None), (32, 17, range(8), None),
         (32, 31, range(9), None), (32, 33, range(4), None), (32, 64, range(10), None), (32, 65, range(7), None),
         (32, 96, range(17), None), (32, 97, range(4), None), (32, 130, range(16), None), (32, 200, range(5), None),
         (24, 20, range(6), "2"), (128, 20, [19, 2, 4, 11], "1"), (128, 66, range(9), "1"), (192, 20, [19, 2, 4, 11], "1")]


@pytest.mark.parametrize("n,nc,nu1,kchunks", CASES)
def test_widths_give_the_same_bits(monkeypatch, n, nc, nu1, kchunks):
    need_gpu()
    nu1 = None if nu1 is None else list(nu1)
    if kchunks:
        monkeypatch.setenv("BS_MABS_KCHUNKS", kchunks)
    V = synth.make_cube(synth.small_workload(n, nc), seed=nc)
    print(f"[narrow widths] n={n} nc={nc} nu1={nu1} kchunks={kchunks}", flush=True)
    c = Ctx()
    h, ncand = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, np.geomspace(1.0, synth.default_umax(n) + 1.0, 4))
    try:
        got = []
        for nj in ("0", "1", "2", "3"):
            monkeypatch.setenv("BS_MABS_NJ", nj)
            got.append(run_gpu(c.h, h, V, bs.BS_SPLIT_BF16, ncand, len(nu1) if nu1 else nc, nc, nu1=nu1))
    finally:
        bs.bs_free_bins(h)
        c.close()
    assert np.all(np.isfinite(got[0][0][got[0][1] > 0]))
    for B, N in got[1:]:
        assert np.array_equal(N, got[0][1])
        assert np.array_equal(B, got[0][0], equal_nan=True)
