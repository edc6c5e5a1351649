"""Residual measurements written over the images they are formed from (X, the
mean image, or both), which the library accepts: the same values, bit for bit,
as with an output of its own.  Sizes where measurements and images take the
same memory, where they take more or less, and several column tiles."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


@pytest.mark.parametrize("nx,ny,nc,q,kind,lm", [(64, 32, 4, 5, "lines", 8), (256, 64, 3, 2, "lines", 40),
                                                (16, 16, 2, 7, "lines", 5), (32, 64, 4, 5, "index", 512),
                                                (64, 64, 3, 4, "index", 3000), (512, 8, 2, 3, "lines", 4)])
def test_residual_over_its_inputs(nx, ny, nc, q, kind, lm):
    cs = Case(datagen.make_small(nx, ny, nc, q, 1, seed=5, kind=kind, n_lines=lm, m=lm, lowrank=False))
    ctx = cs.gpu_ctx()
    n, ny_ = nx * ny, q * nc * int(cs.y.shape[2])
    rng = np.random.default_rng(1)
    Xh = torch.from_numpy(datagen.crandn(rng, q, n).astype(np.complex64))
    zh = torch.from_numpy(datagen.crandn(rng, n).astype(np.complex64))
    X, z = Xh.cuda(), zh.cuda()
    for use_x, use_z in ((True, False), (True, True), (False, True)):
        want = ctx.residual(z if use_z else None, X if use_x else None).clone()
        buf = torch.empty(max(ny_, (q + 1) * n), dtype=torch.complex64, device="cuda:0")
        xb, zb = buf[: q * n].view(q, n), buf[q * n: (q + 1) * n] if use_x else buf[:n]
        if use_x:
            xb.copy_(X)
        zb.copy_(z)
        out = buf[:ny_].view(q, nc, -1)
        ctx.residual(zb if use_z else None, xb if use_x else None, out)
        log(f"  {nx} x {ny} {kind}, X {use_x}, mean {use_z}: equal {bool(torch.equal(out, want))}")
        assert torch.equal(out, want)
