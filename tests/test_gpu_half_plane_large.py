"""test_gpu_half_plane.py's comparison with the FP64 oracle at the sizes it leaves out:
N = 128, and N = 2048 and 4096, where the adjoint's column transforms work by the
two parities of ky (k_half_icols; FP64 at 4096 with two columns per workgroup)
and, in FP32, the forward columns in two passes. Same inputs (windows on both sides of
ku = 0 and across the Nyquist column) and tolerances: FP64 1e-11; FP32 Phi and
Phi^dagger 5e-6, gradient 1e-5."""
import pytest

torch = pytest.importorskip("torch")
import test_gpu_half_plane as H  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("N", [128, 2048, 4096])
def test_half_plane_operator_at_other_sizes(N, prec):
    H.test_half_plane_operator(N, prec)
