"""The SARA dictionary's level kernels at the edges of their tiles, against the
FP64 oracle: a level block of one tile, of less than one (N = 16 has blocks of 2,
4, 8 and 16 elements a side), of several, and the sizes at which the strips per
tile and the split over the bases change (32 .. 1024; 2048 and 4096 are in
test_gpu_sara.py). The caller's buffers start one element off a 16-byte boundary.

Tolerance: a coefficient passes at most eight one-dimensional transforms of at
most 16 fused multiply-adds, each transform orthonormal, so the relative l2
error stays below 8 * 16 * 2^-24 = 7.6e-6 (FP32) and 8 * 16 * 2^-53 (FP64); the
oracle's own FP64 sums round as often again, hence 2x in FP64."""
import numpy as np
import pytest

from _cases import rel
from oracle import sara as S

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _off_by_one(shape, dtype):
    return torch.empty(int(np.prod(shape)) + 1, dtype=dtype, device=DEV)[1:].view(shape)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n", [16, 32, 128, 256, 512, 1024])
def test_level_kernels_match_oracle(n, prec):
    dt = torch.float32 if prec == 32 else torch.float64
    tol = 8 * 16 * 2.0 ** -24 if prec == 32 else 2 * 8 * 16 * 2.0 ** -53
    ctx = R.ri_create(R.plan_desc(n, 0, hmax=0, precision=prec, g_mode=R.RI_G_OTF, tile=16), np.zeros((0, 3)))
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, n)).astype(np.float32).astype(np.float64)
    cr = rng.standard_normal((9, n, n)).astype(np.float32).astype(np.float64)
    xt, out, coef = _off_by_one((n, n), dt), _off_by_one((n, n), dt), _off_by_one((9, n, n), dt)
    xt.copy_(torch.from_numpy(x))
    R.ri_sara_analysis(ctx, xt, coef)
    ref = S.Sara().adj(x)
    for b in range(9):
        assert rel(coef[b].cpu().numpy(), ref[b]) <= tol, b
    coef.copy_(torch.from_numpy(cr))
    R.ri_sara_synthesis(ctx, coef, out)
    assert rel(out.cpu().numpy(), S.Sara().syn(cr)) <= tol
    assert np.array_equal(coef.cpu().numpy(), cr.astype(np.float32 if prec == 32 else np.float64))
