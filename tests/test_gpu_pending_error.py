"""Outputs that a call writes whether or not a device error is pending (a mask
entry out of range, found when the problem is bound): the mean image and the
modelling errors start from zero and stay there."""
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
