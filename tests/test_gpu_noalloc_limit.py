"""The size that ri_gradient_noalloc states where it refuses a context: at N' = 8192 in
FP32 the forward transform keeps its N packed band rows behind the half-plane
output grid, 16 N' cells past the plane, and they count (the call is refused
before any launch)."""
import re

import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_packed_band_counts():
    N, M = 4096, 64
    Np = 2 * N
    ctx = R.ri_create(R.plan_desc(N, M, g_mode=R.RI_G_OTF, hmax=0, tile=16), synth.random_uvw(M, 2.0, 0.0, seed=1))
    x = torch.zeros((N, N), dtype=torch.float32, device=DEV)
    with pytest.raises(R.RIError) as e:
        R.ri_gradient_noalloc(ctx, x, "none", torch.empty_like(x))
    assert e.value.status == R.RI_EINVAL
    need = int(re.search(r"needs (\d+) B", str(e.value)).group(1))
    grid_a, grid_b = 8 * (Np * Np + 16 * Np), 8 * Np * Np
    assert grid_a + grid_b <= need <= grid_a + grid_b + (1 << 17)     # the counter and the partial sums
