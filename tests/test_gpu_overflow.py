"""The first step size where the gradient's FP32 Gram overflows (measurements
of order 1e12 and more: the gradient is of the order of their square, its Gram
of their fourth power): the iteration reports a factor that is not positive
definite.  It must not pass for a stationary start, which ends without a step
and without an error.  The mixed form's FP64 Gram does not overflow and gives
the iterates of the unscaled problem."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, from_gpu_U, log, proj_dist, to_gpu_U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import paper_2212_09664_amd as ag


@pytest.mark.parametrize("r", [3, 8, 11])
def test_overflowing_gradient_is_an_error(r):
    p = datagen.make_small(32, 32, 4, 24, r, seed=90 + r, kind="lines", n_lines=14, lowrank=True, snr_db=30.0)
    cs = Case(p)
    U0 = np.linalg.qr(datagen.crandn(np.random.default_rng(r), p.n, r))[0]
    U1 = to_gpu_U(U0)
    ctx = cs.gpu_ctx(precision=1)
    ctx.init_from(U1)
    _, done = ctx.iterate(2, U1, sync=True)
    assert done == 2
    cs.y32 = (cs.y32 * np.float32(1e13)).astype(np.complex64)
    ctx = cs.gpu_ctx(precision=1)
    U2 = to_gpu_U(U0)
    ctx.init_from(U2)
    _, done = ctx.iterate(2, U2, sync=True)
    d = proj_dist(from_gpu_U(U2), from_gpu_U(U1))
    log(f"  r {r}: mixed form, scaled against not: projectors {d:.1e}")
    assert done == 2 and d < 1e-4
    ctx = cs.gpu_ctx()
    U = to_gpu_U(U0)
    ctx.init_from(U)
    with pytest.raises(ag.AltGDminError) as e:
        ctx.iterate(2, U, sync=True)
    assert e.value.status == 4
