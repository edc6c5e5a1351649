"""The per-line Gram at the edges of its layout, through the LS step's
coefficients: readout lengths below, at and above its 16-row steps (8 leaves two
of the four waves without rows), ranks on either side of its two operand forms
(1, 7, 8 | 9, 15, 16), coil groups with a remainder, lines with fewer and with
more samples than a tile of 8, in both precisions.

Tolerance: b = G^-1 h with G and h sums of products of W, whose FP32
transform errs by 2^-24 a stage (below 2^-22 for these sizes); FP32 sums of
K = nc nx lines products add a rounding walk of 4 sqrt(K) 2^-24.  Both are
amplified by at most twice the condition number of G."""
import numpy as np
import pytest

import datagen
from oracle import altgdmin as AG

from gpu_cases import GPU_OK, Case, from_gpu_B, from_gpu_U, log, rel

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "mixed"])
@pytest.mark.parametrize("nx,ny,nc,q,r", [(8, 32, 5, 6, 1), (8, 16, 3, 21, 4), (16, 32, 4, 20, 7), (16, 16, 7, 40, 9),
                                          (32, 32, 3, 12, 8), (32, 32, 5, 18, 16), (64, 32, 17, 9, 3),
                                          (256, 16, 5, 20, 9), (512, 16, 3, 16, 15)])
def test_ls_step(nx, ny, nc, q, r, precision):
    lines = max(5, ny // 3)
    p = datagen.make_small(nx, ny, nc, q, r, seed=400 + nx + r, kind="lines", n_lines=lines, lowrank=True, snr_db=30.0,
                           variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx(precision=precision)
    U = ctx.init()
    B = from_gpu_B(ctx.gradient(U)[0])
    U0 = from_gpu_U(U)
    ref = AG.ls_step(cs.op, U0, cs.y)
    cond = max(np.linalg.cond(np.stack([cs.op.A(k, U0[:, j]).reshape(-1) for j in range(r)], axis=1)) ** 2
               for k in range(q))
    tol = 2 * cond * (2.0 ** -22 + (4 * np.sqrt(nc * nx * lines) * 2.0 ** -24 if precision == 0 else 0.0))
    e = rel(B, ref)
    log(f"  {nx} x {ny}, {nc} coils, q {q}, r {r}, precision {precision}: {e:.1e} (cond {cond:.1f}, below {tol:.1e})")
    assert e < tol
