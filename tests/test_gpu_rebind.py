"""The gradient where a context is bound to a densely sampled problem, used, and
bound again in the same workspace to one that leaves half of the phase-encode
lines unsampled: the adjoint reads a cleared row for those, not what the first
problem left there (grids and folds as in test_gpu_unsampled, with its
tolerance)."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, log
from test_gpu_unsampled import _gradient_error

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch
    import paper_2212_09664_amd as ag


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "mixed"])
@pytest.mark.parametrize("nx,ny,r", [(32, 16, 2), (8, 32, 3), (16, 64, 3), (32, 128, 5), (16, 256, 9)])
def test_sparse_after_dense(nx, ny, r, precision):
    q, L, dev = 10, ny // 4, torch.device("cuda:0")
    ctx = None
    for dense in (True, False, True):
        p = datagen.make_small(nx, ny, 5, q, r, seed=7 + ny, kind="lines", n_lines=L, lowrank=False, snr_db=30.0,
                               coils="random")
        m = ny if dense else ny // 2
        p.masks = [np.sort([(k * L + i) % m for i in range(L)]).astype(np.int32) for k in range(q)]
        used = len(np.unique(np.concatenate(p.masks)))
        assert used == ny if dense else used == ny // 2
        cs = Case(p)
        if ctx is None:
            ctx = ag.AltGDmin(nx, ny, p.nc, q, r, int(cs.y.shape[2]), 0, precision)
        ws = ctx._keep[4] if ctx._keep else torch.full((ctx.workspace_bytes // 4 + 64,), float("nan"),
                                                       device=dev).view(torch.uint8)
        ctx.set_problem(torch.from_numpy(cs.coils.astype(np.complex64)).to(dev), torch.from_numpy(cs.mask).to(dev),
                        torch.from_numpy(cs.m_k).to(dev), torch.from_numpy(cs.y32).to(dev), workspace=ws)
        e = _gradient_error(ctx, cs, r, ny)
        log(f"  {nx} x {ny}, r {r}, precision {precision}: {used} lines sampled: {e:.1e}")
        assert e < 1e-5
