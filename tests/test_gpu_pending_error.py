"""Outputs that a call writes whether or not a device error is pending (a mask
entry out of range, found when the problem is bound): the mean image and the
modelling errors start from zero and stay there, and a warm start's basis that
cannot be factored (or not for the pending error) is handed back as it came."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


@pytest.mark.parametrize("kind", ["lines", "index"])
@pytest.mark.parametrize("nx,ny", [(16, 16), (8, 64), (128, 32)])
def test_images_are_zero(nx, ny, kind):
    cs = Case(datagen.make_small(nx, ny, 2, 3, 2, seed=0, kind=kind, n_lines=6, m=90))
    cs.mask[1, 0] = nx * ny
    ctx = cs.gpu_ctx()
    y = torch.from_numpy(cs.y32).cuda()
    new = lambda *s: torch.full(s, 7.0, dtype=torch.complex64, device="cuda:0")
    z = ctx.mean(1e-3, 3, new(nx * ny))
    z2 = new(nx * ny)
    ctx.mean_noalloc(z2, 1e-3, 3)
    e1 = ctx.mec_cgls(y, 3, 1e-36, new(3, nx * ny))
    e2 = ctx.mec_ista(y, 3, 1e-3, 0.0, new(3, nx * ny))
    log(f"  {nx} x {ny} {kind}: largest {[float(v.abs().max()) for v in (z, z2, e1, e2)]}")
    assert not any(v.any() for v in (z, z2, e1, e2))
    assert ctx.last_error() == (1, 1)


@pytest.mark.parametrize("r", [2, 7, 12, 16])
@pytest.mark.parametrize("why", ["pending", "zero", "nan"])
def test_basis_is_handed_back(why, r):
    cs = Case(datagen.make_small(16, 32, 2, 3, r, seed=0, kind="lines", n_lines=6))
    if why == "pending":
        cs.mask[1, 0] = 99
    ctx = cs.gpu_ctx()
    U0 = datagen.crandn(np.random.default_rng(r), r, 512).astype(np.complex64)
    if why == "zero":
        U0[:] = 0
    if why == "nan":
        U0[r - 1, 5] = np.nan
    U0 = torch.from_numpy(U0).cuda()
    U = ctx.init_from(U0, torch.full_like(U0, 7.0))
    st, _ = ctx.last_error()
    log(f"  {why}, r {r}: status {st}")
    assert st == (1 if why == "pending" else 4)
    assert torch.equal(torch.view_as_real(U).nan_to_num(-1.0), torch.view_as_real(U0).nan_to_num(-1.0))
