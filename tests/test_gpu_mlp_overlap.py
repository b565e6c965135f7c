"""bs_mlp_predict with y inside the buffer of X gives what it gives into a buffer of its own."""
import pytest

from paper_2506_10526_amd import bs

from gpu_common import Ctx, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [5, 65536])
def test_y_inside_x(n, bf16):
    need_gpu()
    c = Ctx()
    m = bs.bs_mlp_create(c.h, 3, n)
    g = torch.Generator(device="cuda").manual_seed(n)
    X = -6 * torch.rand(n, 4, generator=g, device="cuda")
    try:
        bs.bs_mlp_set_data(m, X, X[:, 0].contiguous())
        ref = torch.empty(n, device="cuda")
        bs.bs_mlp_predict(m, X, ref, bf16=bf16)
        for off in (0, n, 3 * n, 4 * n - 1):   # the last overlaps by one value
            buf = torch.empty(5 * n, device="cuda")
            buf[:4 * n] = X.ravel()
            y = buf[off:off + n]
            bs.bs_mlp_predict(m, buf[:4 * n].view(n, 4), y, bf16=bf16)
            torch.cuda.synchronize()
            assert torch.equal(y, ref), off
    finally:
        bs.bs_mlp_destroy(m)
        c.close()
