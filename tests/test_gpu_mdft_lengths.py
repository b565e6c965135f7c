"""Eq. (dft) at the lengths with a compile-time transform, and their neighbours without one.

Against the FP64 oracle, in both collapse layouts, with fewer line groups than the eight the groups are
dealt in, and with a number that leaves the last part short.  Tolerance: that of the other lengths' test
(1e-12 of max |out|; FP64 FFTs of order eps log2(nc)).
"""
import numpy as np
import pytest

from oracle import estimator as oe
from paper_2506_10526_amd import bs, synth

from gpu_common import Ctx, cuda, host, torch

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("nc,nt", [(32, 3), (64, 1), (64, 9), (72, 2), (96, 5), (128, 3), (144, 3), (192, 2), (216, 2),
                                   (256, 3), (288, 2), (384, 2), (512, 1), (576, 1), (648, 1), (768, 2), (1024, 1)])
@pytest.mark.parametrize("circular", [False, True])
def test_mdft_lengths(nc, nt, circular):
    B = synth.collapsed_mabs(nt, nc, 300 + nc, circular=circular)
    print(f"[mdft] nc={nc} nt={nt} circular={circular}", flush=True)
    c = Ctx()
    out = torch.full((nt, nc, nc), float("nan"), dtype=torch.complex128, device="cuda")
    bs.bs_mabs_dft(c.h, nc, cuda(B), out, scale=0.75, circular=circular)
    got = host(out)
    c.close()
    ref = oe.mabs_dft(B, 0.75, circular=circular)
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref))
