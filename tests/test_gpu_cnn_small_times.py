"""Small images through the denoiser. A network of ten layers without training buffers
skips storing its last hidden layer and takes no longer than the forward pass
of one with them: 0.93 times at 256^2 before layers walked their blocks in alternating
directions, 1.15 times with every second layer backwards at every size (each block then
came from another XCD's L2), and the bound between them."""
import pytest

torch = pytest.importorskip("torch")
import paper_2207_11336_amd.ri as R  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _forward_us(B, h, w, layers, training):
    net = R.ri_cnn_create(layers=layers, max_batch=B, max_h=h, max_w=w, training=training)
    z = torch.randn((B, h, w), device=DEV)
    out = torch.empty_like(z)
    for _ in range(20):
        R.ri_cnn_forward(net, z, out)
    best = []
    for _ in range(9):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(40):
            R.ri_cnn_forward(net, z, out)
        e1.record()
        torch.cuda.synchronize()
        best.append(e0.elapsed_time(e1) / 40 * 1e3)
    net.close()
    return sorted(best)[4]


@pytest.mark.parametrize("B,side", [(1, 256), (16, 64)])
def test_inference_takes_no_longer_than_the_training_forward(B, side):
    a, b = _forward_us(B, side, side, 10, False), _forward_us(B, side, side, 10, True)
    print(f"{B} x {side}^2: {a:.1f} us, with training buffers {b:.1f} us")
    assert a < 1.05 * b
