"""The in-place FP64 eta pass at every length it has (half delay grids of 48 to 384 points) against the
two-buffer form, bit for bit, and the delay grid that FP64 estimates run on: the shortest one that closes the same
triangles, 512 and 768 points among them, equal to the full grid."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, host, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nc", [(12, 96), (18, 128), (16, 192), (12, 256), (16, 384), (18, 512), (12, 768), (12, 64)])
def test_fields_equal_two_buffer_form(monkeypatch, n, nc):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(n + nc)
    V = torch.randn((nc, n, n // 2 + 1), generator=g, device="cuda", dtype=torch.complex128)
    edges = 2 * np.pi * np.geomspace(1.0 / n, ((n - 1) // 3 + 0.5) / n, 3)
    c = Ctx()
    h, _ = bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, edges, du_lambda=1.0, r_mpc=float(n), rprime_mpc_per_mhz=1.0,
                           dnu_mhz=float(n) / nc)
    out = []
    try:
        for two in (False, True):
            if two:
                monkeypatch.setenv("BS_3D_FFT_TWO_BUFFERS", "1")
            F = torch.empty((2, nc, n, n), dtype=torch.float64, device="cuda")
            I = torch.empty((2, nc, n, n), dtype=torch.float64, device="cuda")
            bs.bs_filter_fields(c.h, h, V, 1, bs.BS_FP64, F, count_fields=I)
            out.append((host(F), host(I)))
    finally:
        bs.bs_free_bins(h)
        c.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert np.abs(out[0][0]).max() > 0


@pytest.mark.parametrize("nc,eta,M", [(768, 104, 384), (576, 127, 384), (768, 128, 512), (768, 150, 512), (648, 170, 512),
                                      (864, 171, 768), (768, 200, 768), (512, 100, 384), (512, 130, 512)])
def test_delay_grid_of_fp64_estimates(monkeypatch, nc, eta, M):
    """H = eta on the shortest grid M > 3 H: M as bs_last_timing reports it, counts bit for bit and B within
    1e-12 of B_abs of the full grid's (the rounding of two FP64 transforms and sums)."""
    need_gpu()
    n = 12
    edges = np.array([1.0, 0.3 * eta, 0.7 * eta, eta + 0.5])
    kw = dict(du_lambda=0.05, r_mpc=2 * np.pi, rprime_mpc_per_mhz=2 * np.pi / nc, dnu_mhz=1.0)
    g = torch.Generator(device="cuda").manual_seed(nc)
    V = torch.randn((nc, n, n // 2 + 1), generator=g, device="cuda", dtype=torch.complex128)
    out = []
    for full in (False, True):
        if full:
            monkeypatch.setenv("BS_3D_FULLGRID", "1")
        c = Ctx()
        h, nt = bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, edges, **kw)
        try:
            assert bs.bs_bins_info(h)[0] == eta
            bs.bs_set_timing(c.h, 1)
            B = torch.empty(nt, dtype=torch.float64, device="cuda")
            N = torch.empty(nt, dtype=torch.int64, device="cuda")
            bs.bs_estimate_3d(c.h, h, V, bs.BS_FP64, B, N)
            torch.cuda.synchronize()
            assert bs.bs_last_timing(c.h)[3] == (nc if full else M)
            F = torch.empty((3, nc, n, n), dtype=torch.float64, device="cuda")
            bs.bs_filter_fields(c.h, h, V, 1, bs.BS_FP64, F)
            out.append((host(B), host(N)))
            Fa, tri = F.abs().reshape(3, -1), bs.bs_bins_triangles(h, nt, 3)[0]
            mag = np.array([float((Fa[i] * Fa[j] * Fa[k]).sum()) for i, j, k in tri]) * nc * n * n
        finally:
            bs.bs_free_bins(h)
            c.close()
    assert np.array_equal(out[0][1], out[1][1])
    ok = out[0][1] > 0
    assert ok.any()
    assert np.all(np.abs(out[0][0][ok] - out[1][0][ok]) <= 1e-12 * mag[ok] / out[0][1][ok])
