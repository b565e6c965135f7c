"""The generator at the lengths of its compile-time transforms, and beside them, with strong and with no
non-Gaussianity (the quadratic term is formed about sigma^2 and the sample mean taken out of the cell q =
0 of each channel afterwards) and flagged channels, against the oracle's generator.

Tolerances: FP32 transforms of at most 2^20 points, 5e-7 of the rms of |V| per transform stage group
(2e-6 overall) for every cell; the q = 0 cells are held to the same bar relative to their own size."""
import numpy as np
import pytest

from oracle import generator as og
from paper_2506_10526_amd import bs

from gpu_common import Ctx, cuda, host, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("n,nc", [(48, 96), (64, 128), (96, 192), (128, 96), (192, 24), (36, 256), (24, 384), (16, 512),
                                  (12, 576), (8, 768), (32, 48)])
@pytest.mark.parametrize("f_ng,sigma,flags", [(0.5, 0.5, False), (2.0, 1.5, True), (0.0, 0.5, True)])
def test_cube_matches_oracle(ctx, n, nc, f_ng, sigma, flags):
    cw = np.ones(nc)
    if flags:
        cw[::5] = 0.0
    print(f"[gen lengths] n={n} nc={nc} f={f_ng} sigma={sigma} flags={flags}", flush=True)
    V = torch.empty((nc, n, n // 2 + 1), dtype=torch.complex64, device="cuda")
    bs.bs_generate_cube(ctx, bs.field_desc(n, nc, sigma=sigma, f_ng=f_ng), 9, 4, V, chan_w=cuda(cw, np.float32) if flags else None)
    Vg = host(V).astype(np.complex128)
    Vr = og.generate_cube(n, nc, "cubic", 9, 4, sigma=sigma, f=f_ng, chan_w=cw if flags else None)
    rms = np.sqrt(np.mean(np.abs(Vr) ** 2))
    assert np.all(np.abs(Vg - Vr) <= 2e-6 * np.maximum(np.abs(Vr), rms) * np.log2(n * n * nc))
    assert np.linalg.norm(Vg - Vr) <= 2e-6 * np.linalg.norm(Vr)
    if flags:
        assert np.all(Vg[cw == 0] == 0)
