"""The column transforms of whole planes at every side they are built for: out of
place forwards and backwards (two w-stacks, whose images are complex) in both
precisions, against the FP64 oracle of the same discrete operator; the
in-place FP32 form runs in test_gpu_half_plane.py. Tolerances as there
(relative l2: FP64 1e-11; FP32 5e-6), twice that for the two stacks' sum."""
import functools
import math

import numpy as np
import pytest

import synth
from _cases import rel
from oracle import wstack as WS

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@functools.lru_cache(maxsize=None)
def _case(N, M=607):
    cell = 30 * synth.ARCSEC * 64 / N
    W = 2 * 4.0 / (2 * N * N * cell ** 2)
    uvw = synth.random_uvw(M, 0.999 * math.pi, W, seed=N)
    so = WS.StackedOperator(N, uvw, cell, W, 65, 2)
    x = synth.random_image(N, 5, positive=False).astype(np.float32).astype(np.float64)
    y = (synth.noise_normals(M, 9) * N).astype(np.complex64).astype(np.complex128)
    return uvw, cell, W, x, y, so.phi(x), so.phi_adj(y)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("N", [16, 32, 64, 128, 256, 512, 1024])
def test_stacked_planes(N, prec):
    uvw, cell, W, x, y, phi_x, adj_y = _case(N)
    ctx = R.ri_create(R.plan_desc(N, len(uvw), cell_rad=cell, w_max=W, n_wplanes=65, precision=prec,
                                  g_mode=R.RI_G_OTF, n_wstacks=2), uvw)
    rd, cd = (torch.float32, torch.complex64) if prec == 32 else (torch.float64, torch.complex128)
    xg, yg = torch.tensor(x, dtype=rd, device=DEV), torch.tensor(y, dtype=cd, device=DEV)
    v, a = torch.zeros_like(yg), torch.zeros_like(xg)
    R.phi_forward(ctx, xg, v)
    R.phi_adjoint(ctx, yg, a)
    tol = 2 * (5e-6 if prec == 32 else 1e-11)
    assert rel(v.cpu().numpy(), phi_x) <= tol
    assert rel(a.cpu().numpy(), adj_y) <= tol
