"""The warm-start network in batches large enough for the convolution's tiles
of 256 pixels (more than 1,024 tiles of 64), in each of their shapes with
remainders: 64 x 4, 32 x 8 and 16 x 16.  Reference and tolerances: those of
test_gpu_cnn.test_forward_loss_and_gradients_match_oracle; and both tile sizes
add an output's products in the same order, so that a sequence on its own (the
small tiles) gives the same output bit for bit."""
import pytest

from gpu_cases import GPU_OK, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch
    import paper_2212_09664_amd as ag

CASES = [
    # nx, ny, q, r, width, batch
    (128, 72, 3, 2, 8, 8),
    (88, 88, 17, 2, 8, 8),
    (72, 80, 3, 9, 20, 11),
]


@pytest.mark.parametrize("cfg", CASES, ids=[f"{c[0]}x{c[1]}_b{c[5]}" for c in CASES])
def test_large_batches(cfg):
    from test_gpu_cnn import _data, test_forward_loss_and_gradients_match_oracle as check
    check(cfg)
    nx, ny, q, r, width, batch = cfg
    X, _, p = _data(nx, ny, q, r, width, batch, 1)
    net = ag.WsInit(nx, ny, q, r, width=width, batch=batch)
    X, p = torch.from_numpy(X).cuda(), torch.from_numpy(p).cuda()
    M = net.forward(p, X).clone()
    same = [torch.equal(net.forward(p, X[b:b + 1].contiguous())[0], M[b]) for b in range(batch)]
    log(f"  {cfg}: equal on its own: {same}")
    assert all(same)
