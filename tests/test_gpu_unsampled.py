"""The gradient where some phase-encode lines are sampled by no frame, and
where every line is sampled: the adjoint transforms read the row past the
sampled ones for those that are not, which the fold clears.  The workspace is
poisoned with NaN first, so a row that was not cleared would show.  Grids:
the coil-grouped adjoint (16, 32; any size in the mixed form) and the fused
one (64, 128).  Fold: matrix cores from 16 columns on, else registers.

Tolerance: the gradient is a sum of FP32 transforms and folds, each below
2^-22 of the larger of its two terms, with b from FP32 Grams (below 1e-6 here);
1e-5 is the bound the other gradient tests use."""
import numpy as np
import pytest

import datagen
from oracle import altgdmin as AG

from gpu_cases import GPU_OK, Case, from_gpu_U, log, to_gpu_U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


def _gradient_error(ctx, cs, r, seed):
    U, _ = np.linalg.qr(datagen.crandn(np.random.default_rng(seed), cs.prob.n, r))
    U = U.astype(np.complex64).astype(np.complex128)
    G = from_gpu_U(ctx.gradient(to_gpu_U(U))[1])
    Bref = AG.ls_step(cs.op, U, cs.y)
    Gref = AG.gradient(cs.op, U, Bref, cs.y)
    t1 = np.linalg.norm(AG.gradient(cs.op, U, Bref, np.zeros_like(cs.y)))
    t2 = np.linalg.norm(AG.gradient(cs.op, np.zeros_like(U), Bref, cs.y))
    return np.linalg.norm(G - Gref) / max(t1, t2)


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "mixed"])
@pytest.mark.parametrize("nx,ny,r", [(32, 16, 2), (8, 32, 3), (16, 64, 3), (32, 128, 5)])
def test_gradient(nx, ny, r, precision):
    # a dense mask, then a sparse one of the same shapes
    lines = [ny - 1, ny // 4]
    cases = []
    for i, nl in enumerate(lines):
        p = datagen.make_small(nx, ny, 5, 6 if i else 8, r, seed=700 + ny + i, kind="lines", n_lines=nl, lowrank=False,
                               snr_db=30.0, coils="random")
        cases.append(Case(p))
    for cs in cases:
        p = cs.prob
        import paper_2212_09664_amd as ag
        ctx = ag.AltGDmin(p.nx, p.ny, p.nc, p.q, p.r, int(cs.y.shape[2]), 0, precision)
        ws = torch.full((ctx.workspace_bytes // 4 + 64,), float("nan"), device="cuda:0").view(torch.uint8)
        dev = torch.device("cuda:0")
        ctx.set_problem(torch.from_numpy(cs.coils.astype(np.complex64)).to(dev), torch.from_numpy(cs.mask).to(dev),
                        torch.from_numpy(cs.m_k).to(dev), torch.from_numpy(cs.y32).to(dev), workspace=ws)
        e = _gradient_error(ctx, cs, r, ny)
        used = len(np.unique(cs.mask[cs.mask >= 0]))
        log(f"  {nx} x {ny}, r {r}, precision {precision}: {used} of {ny} lines sampled: {e:.1e}")
        assert e < 1e-5
