"""Parameter gradients of the CNN at the edges of the weight-gradient blocks (32 x 8
pixels, two per workgroup): sides that leave half a block, a single pair of
blocks, more pairs than workgroups deal evenly. The network of
test_gpu_cnn_exact.py, whose sums are exact in FP32 in any order (checked on the
CPU there and here), so the gate is its 1e-6 relative l2."""
import numpy as np
import pytest

from _cases import rel
from oracle import cnn as OC
from test_gpu_cnn_exact import L, _check_exact_backward, _check_exact_forward, _dyadic, _exact_net

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,h,w", [(1, 16, 16), (3, 16, 48), (1, 48, 32), (2, 32, 80), (9, 16, 16)])
def test_parameter_gradients_exact(B, h, w):
    params = _exact_net(5)
    z, g = _dyadic((B, h, w), 6, 0, 32), _dyadic((B, h, w), 7, -8, 9)
    _, acts = OC.forward(params, z, bf16=True)
    _check_exact_forward(params, acts)
    _check_exact_backward(params, acts, g)
    ref = OC.backward(params, acts, g, bf16=True)
    vec = np.concatenate([np.concatenate([w_.ravel(), b_.ravel()]) for w_, b_ in params]).astype(np.float32)
    net = R.ri_cnn_create(layers=L, max_batch=B, max_h=h, max_w=w, training=True)
    R.ri_cnn_set_params(net, torch.tensor(vec, device=DEV))
    grads = torch.empty(net.n_params, dtype=torch.float32, device=DEV)
    R.ri_cnn_grad(net, torch.tensor(z, dtype=torch.float32, device=DEV),
                  torch.tensor(g, dtype=torch.float32, device=DEV), grads)
    want = np.concatenate([np.concatenate([dw.ravel(), db.ravel()]) for dw, db in ref])
    got = grads.cpu().numpy().astype(np.float64)
    o = 0
    for dw, db in ref:
        for r in (dw, db):
            e = rel(got[o:o + r.size], want[o:o + r.size])
            assert e <= 1e-6, e
            o += r.size
