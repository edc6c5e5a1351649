"""The operator and its adjoint where the columns are short (8, 16 and 32 rows),
over coil counts around the groups of threads that take the coils side by
side (4 or 8), with images narrower and wider than a column tile.

Tolerance: 2 log2 N roundings a transform (at most 9 + 5 stages), the coil's
product, and for the adjoint a sum over up to 17 coils, each 2^-24 of a term at
most: below 50 * 2^-24 = 3e-6."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, log, rel

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


@pytest.mark.parametrize("kind", ["lines", "index"])
@pytest.mark.parametrize("nc", [1, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("nx,ny", [(8, 8), (8, 16), (64, 16), (16, 32), (512, 8), (128, 32)])
def test_operator_and_adjoint(nx, ny, nc, kind):
    p = datagen.make_small(nx, ny, nc, 3, 1, seed=nc, kind=kind, n_lines=ny // 2, m=nx * ny // 3, lowrank=False,
                           coils="random", variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx()
    x32 = datagen.crandn(np.random.default_rng(nc), p.n, p.q).astype(np.complex64)
    Y = ctx.apply_A(torch.from_numpy(np.ascontiguousarray(x32.T)).cuda()).cpu().numpy()
    X = ctx.apply_AH(torch.from_numpy(cs.y32).cuda()).cpu().numpy().T
    ea = rel(Y.astype(np.complex128), cs.op.apply_A(x32.astype(np.complex128)))
    eh = rel(X.astype(np.complex128), cs.op.apply_AH(cs.y))
    log(f"  {nx} x {ny}, {nc} coils, {kind}: A {ea:.1e}, A^H {eh:.1e}")
    assert ea < 3e-6 and eh < 3e-6
