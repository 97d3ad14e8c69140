"""The SARA dictionary with the image inside the coefficients: on one of the wavelet
planes, across two of them, and (synthesis) on the Dirac plane. Same bits as with
buffers of their own, which test_gpu_sara.py and test_gpu_sara_tiles.py compare
with the oracle. 64 and 512 transform the finest level basis by basis, 1024
and 2048 all bases in one workgroup."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n", [64, 512, 1024, 2048])
def test_in_place(n, prec):
    dt = torch.float32 if prec == 32 else torch.float64
    ctx = R.ri_create(R.plan_desc(n, 0, hmax=0, precision=prec, g_mode=R.RI_G_OTF, tile=16), np.zeros((0, 3)))
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    x = torch.randn((n, n), generator=g, device=DEV, dtype=dt)
    c = torch.randn((9, n, n), generator=g, device=DEV, dtype=dt)
    coef, out = torch.empty_like(c), torch.empty_like(x)
    R.ri_sara_analysis(ctx, x, coef)
    R.ri_sara_synthesis(ctx, c, out)
    for at in (n * n, 5 * n * n, 8 * n * n, 2 * n * n + 7 * n):
        buf = torch.empty(9 * n * n, device=DEV, dtype=dt)
        view = buf[at:at + n * n].view(n, n)
        view.copy_(x)
        R.ri_sara_analysis(ctx, view, buf.view(9, n, n))
        assert torch.equal(buf.view(9, n, n), coef), at
    for at in (0, n * n, 5 * n * n, 8 * n * n, 2 * n * n + 7 * n):
        buf = c.flatten().clone()
        view = buf[at:at + n * n].view(n, n)
        R.ri_sara_synthesis(ctx, buf.view(9, n, n), view)
        assert torch.equal(view, out), at
