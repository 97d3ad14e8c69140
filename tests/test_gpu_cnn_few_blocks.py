"""The hidden layers of the denoiser where a launch has one block of pixels per workgroup:
a layer is then the load of its weights (74 KB) and little more. Ten layers against three
at the same size: 4.5 times as long with the weights loaded once per workgroup, 4.9 times
with every wave loading its own (295 KB per workgroup), and the bound between them."""
import pytest

from test_gpu_cnn_small_times import _forward_us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,h,w", [(1, 16, 16), (200, 16, 16)])
def test_a_layer_of_few_blocks_costs_one_load_of_its_weights(B, h, w):
    ten, three = _forward_us(B, h, w, 10, False), _forward_us(B, h, w, 3, False)
    print(f"{B} x {h} x {w}: {ten:.1f} us, three layers {three:.1f} us")
    assert ten < (4.7 if B == 1 else 4.3) * three
