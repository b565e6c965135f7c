"""The compile-time LDS transforms of the 3D field passes against the run-time two-buffer form, which does
the same butterflies in the same order: shell fields equal bit for bit at every length that has a
compile-time transform, with ragged last blocks, in both precisions."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, host, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("n,nc", [(48, 96), (64, 128), (96, 192), (128, 256), (192, 384), (256, 96), (48, 768), (64, 24)])
@pytest.mark.parametrize("prec", [bs.BS_FP32, bs.BS_FP64])
def test_fields_equal_run_time_plan(ctx, monkeypatch, n, nc, prec):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + nc)
    V = torch.randn((nc, n, n // 2 + 1), generator=g, device="cuda", dtype=torch.complex128 if prec == bs.BS_FP64 else torch.complex64)
    edges = 2 * np.pi * np.geomspace(1.0 / n, ((n - 1) // 3 + 0.5) / n, 3)
    print(f"[fft lengths] n={n} nc={nc} prec={prec}", flush=True)
    h, _ = bs.bs_make_bins(ctx, bs.BS_SHELL_K, n, nc, edges, du_lambda=1.0, r_mpc=float(n), rprime_mpc_per_mhz=1.0,
                           dnu_mhz=float(n) / nc)
    out = []
    try:
        for two in (False, True):
            if two:
                monkeypatch.setenv("BS_3D_FFT_TWO_BUFFERS", "1")
            F = torch.empty((2, nc, n, n), dtype=torch.float64 if prec == bs.BS_FP64 else torch.float32, device="cuda")
            bs.bs_filter_fields(ctx, h, V, 1, prec, F)
            out.append(host(F))
    finally:
        bs.bs_free_bins(h)
    assert np.array_equal(out[0], out[1])
