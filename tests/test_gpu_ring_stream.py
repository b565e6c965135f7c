"""Ring fields of a call larger than the last-level cache: the same bits as those of smaller calls.

A channel's fields do not depend on the other channels, and the non-temporal stores of large calls change no
value, so each channel must equal, bit for bit, its fields from a call with a few channels (which the
oracle's tests cover).
"""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nc,prec", [(256, 176, bs.BS_FP32), (128, 700, bs.BS_FP32), (256, 90, bs.BS_FP64),
                                       (96, 1300, bs.BS_FP64)])
def test_large_calls(n, nc, prec):
    cd, rd = (torch.complex128, torch.float64) if prec == bs.BS_FP64 else (torch.complex64, torch.float32)
    g = torch.Generator(device="cuda").manual_seed(n + nc)
    V = torch.randn((nc, n, n // 2 + 1), generator=g, device="cuda", dtype=cd)
    edges = np.geomspace(1.0, (n - 1) // 3, 7)
    print(f"[ring stream] n={n} nc={nc} precision={prec}", flush=True)
    c = Ctx()

    def fields(v):
        v = v.contiguous()
        h, _ = bs.bs_make_bins(c.h, bs.BS_RING_U, n, v.shape[0], edges)
        F = torch.full((6, v.shape[0], n, n), 7.0, dtype=rd, device="cuda")
        bs.bs_filter_fields(c.h, h, v, 0, prec, F, None)
        torch.cuda.synchronize()
        bs.bs_free_bins(h)
        return F

    big = fields(V)
    assert big.numel() * big.element_size() > 1 << 28
    for c0 in (0, nc // 2, nc - 8):
        assert torch.equal(fields(V[c0:c0 + 8]), big[:, c0:c0 + 8])
    c.close()
