"""The row-local training kernel at the edges of its 16-row groups, of its block count (larger
batches loop over 1024 blocks) and of the weight gradients' row splits, against the FP64 oracle.

Tolerances: FP32 products and sums of at most 256 terms a layer and a fixed-order sum over rows;
the relative error of a sum of n FP32 terms stays below about sqrt(n) 2^-24 per factor, 1e-5 for
these sizes (loss) and 2e-5 normwise per parameter group (gradient, three layers deep)."""
import numpy as np
import pytest

from oracle import mlp as om
from paper_2506_10526_amd import bs

from gpu_common import Ctx, cuda, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Ctx()
    yield c.h
    c.close()


@pytest.mark.parametrize("n", [2, 15, 16, 17, 63, 64, 65, 511, 513, 16384, 16400])
def test_loss_grad_and_prediction(ctx, n):
    rng = np.random.default_rng(n)
    X = rng.uniform(-6, 0, (n, 4)).astype(np.float32)
    t = (np.sin(X[:, 0]) + 0.3 * X[:, 1] * X[:, 2]).astype(np.float32)
    print(f"[mlp rows] n={n}", flush=True)
    m = bs.bs_mlp_create(ctx, 3, n)
    try:
        bs.bs_mlp_set_data(m, cuda(X), cuda(t))
        st = bs.bs_mlp_read_state(m).astype(np.float64)
        theta, nm = st[:bs.BS_MLP_NPARAM], st[bs.BS_MLP_NPARAM:]
        xn, tn = (X.astype(np.float64) - nm[:4]) / nm[4:8], (t.astype(np.float64) - nm[8]) / nm[9]
        L_ref, g_ref = om.loss_and_grad(theta, xn, tn)
        g = torch.empty(bs.BS_MLP_NPARAM, dtype=torch.float32, device="cuda")
        L = bs.bs_mlp_loss_grad(m, g)
        assert abs(L - L_ref) <= 1e-5 * L_ref
        gg, o = g.cpu().numpy().astype(np.float64), 0
        for name, shape in om.SHAPES:
            a, o = o, o + int(np.prod(shape))
            err = np.linalg.norm(gg[a:o] - g_ref[a:o]) / max(np.linalg.norm(g_ref[a:o]), 1e-30)
            assert err <= 2e-5, (name, err)
        y = torch.empty(n, dtype=torch.float32, device="cuda")
        bs.bs_mlp_predict(m, cuda(X), y)
        yref = nm[8] + nm[9] * om.forward(theta, xn)
        assert np.allclose(y.cpu().numpy(), yref, rtol=1e-5, atol=1e-5 * max(1.0, np.abs(yref).max()))
    finally:
        bs.bs_mlp_destroy(m)
