"""The 3D counts are certified with the length of the contraction's MFMA runs: a shell whose counts
128-voxel runs cannot certify (and shorter ones can) is summed in shorter ones."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, host, need_gpu, torch

pytestmark = pytest.mark.gpu


def stages(L):
    return 0 if L == 1 else 1 + stages(L // 2) if L % 2 == 0 else 2 + stages(L // 3)


def bound(S, n, nc, run):
    """Error bound of the count of three shells of S cells, runs of `run` voxels, on the full delay grid."""
    vox = nc * n * n
    chunk = -(-(-(-vox // 1024)) // 128) * 128
    depth = run + -(-chunk // 4 // run) + 3 + 32 + -(-(-(-vox // chunk)) // 32)
    eps = 2 * (1 + 4 * np.sqrt(2)) * (2 * stages(n) + stages(nc) + 2) + 3
    return 1.001 * 2.0 ** -53 * (3 * eps + depth + 4) * float(S) ** 2


@pytest.mark.parametrize("n, nc", [(128, 324), (192, 144)])
def test_shell_between_the_run_lengths(n, nc):
    need_gpu()
    umax = 0.48 * n   # closure mod n: the delay grid keeps its nc points
    u, q = np.fft.fftfreq(n, 1.0 / n), np.fft.fftfreq(nc, 1.0 / nc)
    s = (u[:, None] ** 2 + u[None, :] ** 2).ravel()
    s = s[(s >= 1) & (s <= umax ** 2)]
    k2 = np.sort((s[:, None] / n ** 2 + (q[np.abs(q) < nc / 2] / nc)[None, :] ** 2).ravel())
    S = next(x for x in range(1_000_000, k2.size, 1000) if bound(x, n, nc, 128) > 0.505)
    R = np.sqrt(k2[S]) * (1 + 1e-9)
    S = int(np.searchsorted(k2, R * R))
    assert bound(S, n, nc, 128) > 0.5 and min(bound(S, n, nc, r) for r in (64, 32)) < 0.5
    c = Ctx()
    h, nt = bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, [1e-6, 2 * np.pi * R], umax=umax, du_lambda=1.0, r_mpc=float(n),
                            rprime_mpc_per_mhz=1.0, dnu_mhz=1.0)
    try:
        assert nt == 1 and int(bs.bs_bins_triangles(h, nt, 1)[1][0]) == S
        V = torch.zeros((nc, n, n // 2 + 1), dtype=torch.complex64, device="cuda")
        B = torch.empty(1, dtype=torch.float64, device="cuda")
        T = torch.empty(1, dtype=torch.int64, device="cuda")
        bs.bs_estimate_3d(c.h, h, V, bs.BS_FP32, B, T)
        assert bs.bs_last_count_dev(c.h) <= bs.bs_last_count_bound(c.h) < 0.5
        # the count from the same fields in double precision on the host
        ind = np.zeros((nc, n, n))
        uu = u[None, :, None] ** 2 + u[None, None, :] ** 2
        kk = uu / n ** 2 + (q / nc)[:, None, None] ** 2
        ind[(uu >= 1) & (uu <= umax ** 2) & (np.abs(q)[:, None, None] < nc / 2) & (kk < R * R)] = 1.0
        assert int(ind.sum()) == S
        F = np.fft.ifftn(ind).real
        want = float(nc * n * n) ** 2 * float(np.sum(F ** 3, dtype=np.longdouble))
        assert abs(int(host(T)[0]) - want) < 0.5
    finally:
        bs.bs_free_bins(h)
        c.close()
