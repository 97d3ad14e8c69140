"""FP32 visibilities keep their bits whichever kernels form F Z x: one real image goes
in place (at N' = 8192 through the packed band rows), a stack of the w-stacking
hybrid out of place over the whole plane. With a pixel size so small that the phase
screens are 1 and every w at the centre of its stack (no w-kernel), both contexts
hold the same G, and Phi x has to come out equal, not close."""
import math

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N", [16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
def test_same_bits(N):
    M, W = 3001, 1024.0
    x = torch.tensor(synth.random_image(N, 3, positive=False), dtype=torch.float32, device=DEV)
    out = []
    for stacks, w in ((0, 0.0), (2, W / 2)):
        uvw = synth.random_uvw(M, 0.999 * math.pi, 0.0, seed=N)
        uvw[:, 2] = w
        ctx = R.ri_create(R.plan_desc(N, M, cell_rad=1e-30, w_max=W, n_wplanes=65, precision=32, g_mode=R.RI_G_OTF,
                                      tile=8, n_wstacks=stacks), uvw)
        y = torch.zeros(M, dtype=torch.complex64, device=DEV)
        R.phi_forward(ctx, x, y)
        out.append(y.cpu().numpy())
        R.ri_destroy(ctx)
    assert np.linalg.norm(out[0]) > 0
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32)), np.mean(out[0] != out[1])
