"""Calls captured into a graph upload their tables when the graph is replayed, not when they are
captured: eager calls before, between and after the replays, with the same and with other tables, give
what they give without a graph, and so does every replay."""
import numpy as np
import pytest

from paper_2506_10526_amd import bs, synth

from gpu_common import need_gpu, torch, vis_tensor

pytestmark = pytest.mark.gpu


class Streamed:
    """A context on a stream of its own, so that its calls can be captured."""

    def __init__(self):
        self.s = torch.cuda.Stream()
        self.h = bs.bs_create(0, self.s.cuda_stream)

    def run(self, call, out):
        torch.cuda.synchronize()
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        call(out)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    def capture(self, call, out):
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=self.s, capture_error_mode="relaxed"):
            call(out)
        return g

    def replay(self, g, out):
        torch.cuda.synchronize()
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]


def same(a, b):
    return all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b))


def check(c, a, b, out_a, out_b):
    """a and b: calls with different tables of the same sizes."""
    ra, rb = c.run(a, out_a), c.run(b, out_b)
    assert same(c.run(a, out_a), ra)
    cap = [torch.zeros_like(t) for t in out_b]
    g = c.capture(b, cap)
    assert same(c.run(b, out_b), rb)           # the tables of b are not on the device yet
    assert same(c.run(a, out_a), ra)
    for _ in range(3):
        assert same(c.replay(g, cap), rb)
        assert same(c.run(a, out_a), ra)       # the replay left b's tables
        assert same(c.run(b, out_b), rb)


def test_mabs_tables():
    need_gpu()
    n, nc = 16, 6
    c = Streamed()
    h, nt = bs.bs_make_bins(c.h, bs.BS_RING_U, n, nc, np.geomspace(1.0, 6.0, 5))
    tri = bs.bs_bins_triangles(h, nt, 4)[0]
    V = vis_tensor(synth.make_cube(synth.small_workload(n, nc), seed=2), bs.BS_FP64)

    def call(sel, nu1):
        return lambda o: bs.bs_estimate_mabs(c.h, h, V, bs.BS_FP64, o[0], o[1], tri3=sel, nu1=nu1)

    def out():
        return [torch.zeros((nt, 2, nc, nc), dtype=dt, device="cuda") for dt in (torch.float64, torch.int64)]

    try:
        check(c, call(tri, [0, 1]), call(tri[::-1], [3, 2]), out(), out())
    finally:
        torch.cuda.synchronize()
        bs.bs_free_bins(h)
        bs.bs_destroy(c.h)


@pytest.mark.parametrize("prec", [bs.BS_FP64, bs.BS_SPLIT_BF16])
def test_3d_plan(prec):
    """The captured call plans anew: the plan kept by the context is another one."""
    need_gpu()
    n, nc = 16, 32
    c = Streamed()
    V = vis_tensor(synth.make_cube(synth.small_workload(n, nc), seed=4), prec)
    bins, calls, outs = [], [], []
    for hi in (5.5, 4.5):
        h, nt = bs.bs_make_bins(c.h, bs.BS_SHELL_K, n, nc, 2 * np.pi * np.geomspace(1.0 / n, hi / n, 6), du_lambda=1.0,
                                r_mpc=float(n), rprime_mpc_per_mhz=1.0, dnu_mhz=float(n) / nc)
        bins.append(h)
        calls.append(lambda o, h=h: bs.bs_estimate_3d(c.h, h, V, prec, o[0], o[1], o[2]))
        outs.append([torch.zeros(nt, dtype=dt, device="cuda") for dt in (torch.float64, torch.int64, torch.float64)])
    try:
        check(c, calls[0], calls[1], outs[0], outs[1])
    finally:
        torch.cuda.synchronize()
        for h in bins:
            bs.bs_free_bins(h)
        bs.bs_destroy(c.h)
