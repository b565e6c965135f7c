"""The blocks of the FP64 3D contraction: small cubes are spread over the chip (a cube a hundredth of another's
takes less than 0.6 of its time), and counts and estimates agree with the oracle at voxel counts on both sides
of the rule's lines (three slabs a block, 512 blocks, a dozen slabs)."""
import numpy as np
import pytest

from oracle import bins as ob
from oracle import counts as oc
from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, compare_B, host, need_gpu, torch, vis_tensor

pytestmark = pytest.mark.gpu


def bins(c, n, nc, edges):
    return bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, edges, du_lambda=1.0, r_mpc=float(n), rprime_mpc_per_mhz=1.0,
                           dnu_mhz=float(n) / nc)


# 128, 384 +- 128, 512 blocks of three slabs (196,608 voxels) and below and above it
@pytest.mark.parametrize("n,nc", [(8, 2), (8, 4), (8, 6), (8, 8), (16, 32), (48, 96), (64, 48), (64, 54)])
def test_counts_and_estimate(n, nc):
    need_gpu()
    shells = 3
    edges = 2 * np.pi / n * np.linspace(0.9, (n - 1) // 3 + 0.5, shells + 1)
    V = synth.make_cube(synth.small_workload(n, nc), seed=n + nc)
    b = ob.make_bins(ob.SHELL_K, n, nc, edges, du=1.0, r_mpc=float(n), rprime=1.0, dnu=float(n) / nc)
    T, _ = oc.exact_counts(b)
    f = oe.ShellFields(b, V)
    Bref, _, neff, _, _ = oe.estimate_3d(b, V, fields=f, counts=T)
    A = np.array([np.sum(np.abs(f.data(i) * f.data(j) * f.data(k))) for i, j, k in b.triangles])
    scale = np.where(T > 0, nc * n * n * A / np.maximum(neff, 1.0), 0.0)
    c = Ctx()
    h, nt = bins(c, n, nc, edges)
    try:
        B = torch.empty(nt, dtype=torch.float64, device="cuda")
        N = torch.empty(nt, dtype=torch.int64, device="cuda")
        bs.bs_estimate_3d(c.h, h, vis_tensor(V, bs.BS_FP64), bs.BS_FP64, B, N)
        Bg, Ng = host(B), host(N)
    finally:
        bs.bs_free_bins(h)
        c.close()
    assert nt == len(b.triangles) and np.array_equal(Ng, T)
    compare_B(Bg, Bref, T, scale, 1e-10)


def test_small_cubes_are_spread():
    need_gpu()
    c = Ctx()
    bs.bs_set_timing(c.h, True)

    def us(n, nc, shells, top):
        h, nt = bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, 2 * np.pi * np.geomspace(1.0 / n, top, shells + 1),
                                du_lambda=1.0, r_mpc=float(n), rprime_mpc_per_mhz=1.0, dnu_mhz=1.0)
        V = torch.ones((nc, n, n // 2 + 1), dtype=torch.complex128, device="cuda")
        B = torch.empty(nt, dtype=torch.float64, device="cuda")
        N = torch.empty(nt, dtype=torch.int64, device="cuda")
        t = []
        for _ in range(25):
            bs.bs_estimate_3d(c.h, h, V, bs.BS_FP64, B, N)
            torch.cuda.synchronize()
            t.append(1e3 * bs.bs_last_timing(c.h)[1])
        bs.bs_free_bins(h)
        return np.median(t[5:])

    try:
        small, large = us(16, 32, 4, 0.45), us(48, 96, 12, 0.3)
        print(f"[contract64 blocks] 16^2 x 32 {small:.1f} us, 48^2 x 96 {large:.1f} us", flush=True)
        assert small <= 0.6 * large, (small, large)
    finally:
        c.close()
