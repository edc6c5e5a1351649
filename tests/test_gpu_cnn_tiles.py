"""The warm-start network at the edges of its kernels' tiles: images whose
sides are no multiple of the 16-pixel convolution tile or the 32-pixel
weight-gradient block, every class of input channel count (32, 64, 96 per
workgroup, and two workgroups), and ranks in each tile class of the loss's
Gram up to the largest.  Reference and tolerances: those of
test_gpu_cnn.test_forward_loss_and_gradients_match_oracle."""
import pytest

from gpu_cases import GPU_OK

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

CASES = [
    # nx, ny, q, r, width, batch
    (8, 40, 17, 1, 4, 3),
    (40, 24, 33, 16, 32, 1),
    (72, 8, 50, 9, 17, 2),
    (56, 16, 16, 5, 32, 2),
]


@pytest.mark.parametrize("cfg", CASES, ids=[f"{c[0]}x{c[1]}_q{c[2]}_r{c[3]}_w{c[4]}" for c in CASES])
def test_network_over_tile_shapes(cfg):
    from test_gpu_cnn import test_forward_loss_and_gradients_match_oracle as check
    check(cfg)
