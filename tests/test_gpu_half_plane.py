"""The half-plane grids of a real image: Phi, Phi^dagger and the gradient on every
shape of the column passes, with windows on both sides of ku = 0 and across
the Nyquist column, against the FP64 oracle. Tolerances as in
test_gpu_operator.py (relative l2: FP64 1e-11; FP32 Phi and Phi^dagger 5e-6,
gradient 1e-5)."""
import functools
import math

import numpy as np
import pytest

import synth
from _cases import rel
from oracle import phi as OP

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@functools.lru_cache(maxsize=None)
def _case(N, M=1203):
    cell = 30 * synth.ARCSEC * 64 / N
    W = 2 * 4.0 / (2 * N * N * cell ** 2)
    uvw = synth.random_uvw(M, 0.999 * math.pi, W, seed=N)
    cells = np.array([-N, -N + 1, -9, -1, 0, 1, 8, N - 1, N]) * (math.pi / N)   # u cells at the folds
    k = np.arange(M // 3)
    uvw[k, 0] = np.clip(cells[k % 9] + uvw[k, 0] / (10 * N), -0.9999 * math.pi, 0.9999 * math.pi)
    op = OP.Operator(N, uvw, cell=cell, W=W, n_wplanes=65)
    x = synth.random_image(N, 5, positive=False)
    y = synth.noise_normals(M, 9) * N
    return uvw, cell, W, x, y, op.phi(x), op.phi_adj(y), op.grad(x, y)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("N", [16, 32, 64, 256, 512, 1024])
def test_half_plane_operator(N, prec):
    uvw, cell, W, x, y, phi_x, adj_y, (g_ref, r2_ref) = _case(N)
    M = len(uvw)
    ctx = R.ri_create(R.plan_desc(N, M, cell_rad=cell, w_max=W, n_wplanes=65, precision=prec, g_mode=R.RI_G_OTF,
                                  tile=8), uvw)
    rd, cd = (torch.float32, torch.complex64) if prec == 32 else (torch.float64, torch.complex128)
    xg, yg = torch.tensor(x, dtype=rd, device=DEV), torch.tensor(y, dtype=cd, device=DEV)
    v, a, g = torch.zeros_like(yg), torch.zeros_like(xg), torch.zeros_like(xg)
    r2 = torch.zeros(1, dtype=torch.float64, device=DEV)
    R.phi_forward(ctx, xg, v)
    R.phi_adjoint(ctx, yg, a)
    R.ri_set_data(ctx, yg)
    R.ri_gradient(ctx, xg, None, g, r2)
    tol = 5e-6 if prec == 32 else 1e-11
    assert rel(v.cpu().numpy(), phi_x) <= tol
    assert rel(a.cpu().numpy(), adj_y) <= tol
    assert rel(g.cpu().numpy(), g_ref) <= 2 * tol
    assert abs(r2.item() - r2_ref) <= tol * r2_ref
