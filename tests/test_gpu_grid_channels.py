"""Gridding of many baselines on few and on odd numbers of channels: staged and unstaged calls on both sides
of the rule, shares of the baselines that do not divide by the groups that add them, channels past a multiple
of eight, grids whose cells far outnumber the baselines.  Counts bit for bit, FP64 sums within 1e-12 of each
cell's sum of |Re V| + |Im V|.  And fewer channels take no longer than more of them."""
import numpy as np
import pytest

from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nco,nvis", [(256, 1, 70001), (256, 2, 300000), (256, 9, 262144), (256, 17, 140000), (256, 35, 50001),
                                        (64, 3, 50000), (130, 30, 100000), (2048, 3, 33000), (4096, 2, 40000)])
def test_channels(n, nco, nvis):
    need_gpu()
    du = synth.DU_G
    rng = np.random.default_rng(n + nvis)
    uv = rng.uniform(-0.51 * n * du, 0.51 * n * du, (nvis, 2))
    uv[:nvis // 2] *= rng.random((nvis // 2, 1)) ** 3            # half of them crowd around the origin
    uv[:300, 1] = rng.uniform(-0.4 * du, 0.4 * du, 300)          # the line q_v = 0
    vis = (rng.normal(size=(1, nvis)) + 1j * rng.normal(size=(1, nvis))).astype(np.complex64)
    v64 = vis.astype(np.complex128)
    print(f"[grid channels] n={n} nco={nco} nvis={nvis}", flush=True)
    rV, rN = oe.grid_visibilities(uv, v64, None, n, du, 1)
    mag, _ = oe.grid_visibilities(uv, np.abs(v64.real) + np.abs(v64.imag), None, n, du, 1)
    c = Ctx()
    vd = cuda(vis).repeat(nco, 1)
    Vg = torch.full((nco, n, n // 2 + 1), 3.0, dtype=torch.complex128, device="cuda")
    Ng = torch.full((nco, n, n // 2 + 1), 3, dtype=torch.int32, device="cuda")
    bound = cuda(1e-12 * np.abs(mag) + 1e-300)
    try:
        for _ in range(2):
            bs.bs_grid_visibilities(c.h, n, du, cuda(uv), vd, Vg, Ng, chan_avg=1, precision=bs.BS_FP64)
            assert torch.equal(Ng, cuda(rN).to(torch.int32).expand_as(Ng))
            assert bool(((Vg - cuda(rV)).abs() <= bound).all())
            Vg.fill_(5.0)
    finally:
        c.close()


@pytest.mark.parametrize("n,few,more,nvis", [(256, 1, 9, 262144), (2048, 4, 8, 65536), (4096, 1, 2, 262144)])
def test_fewer_channels_take_no_longer(n, few, more, nvis):
    need_gpu()
    uv = cuda(synth.uv_tracks(nvis, 1, 0.6 * synth.DU_G, 0.5 * n * synth.DU_G))
    c = Ctx()

    def us(nco):
        vis = torch.ones((nco, nvis), dtype=torch.complex64, device="cuda")
        V = torch.empty((nco, n, n // 2 + 1), dtype=torch.complex64, device="cuda")
        N = torch.empty((nco, n, n // 2 + 1), dtype=torch.int32, device="cuda")
        t = []
        for _ in range(15):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            bs.bs_grid_visibilities(c.h, n, synth.DU_G, uv, vis, V, N)
            b.record()
            torch.cuda.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        return np.median(t[3:])

    try:
        x, y = us(few), us(more)
        print(f"[grid channels] n={n}: {few} {x:.0f} us, {more} {y:.0f} us", flush=True)
        assert x <= 1.1 * y, (x, y)
    finally:
        c.close()
