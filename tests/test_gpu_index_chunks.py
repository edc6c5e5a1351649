"""General masks where the operators work through the frames in two chunks (a
chunk's coil images fill 256 MiB: 16 frames of 8 coils at 512 x 512; here 18):
the operator and its adjoint bit for bit as over the same frames in one chunk,
MEC-1 and MEC-2 against FP64 references.

Tolerances: test_gpu_normal's (three CGLS iterations, 5e-5; ISTA, 5e-5)."""
import numpy as np
import pytest

import datagen
from oracle import mri as R

from gpu_cases import GPU_OK, Case, log, rel

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch
    import paper_2212_09664_amd as ag


def test_two_chunks_of_frames():
    p = datagen.make_small(512, 512, 8, 18, 1, seed=3, kind="index", m=9000, lowrank=False, variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx()
    dev = torch.device("cuda:0")
    X = torch.from_numpy(datagen.crandn(np.random.default_rng(4), p.q, p.n).astype(np.complex64)).to(dev)
    y = torch.from_numpy(cs.y32).to(dev)
    z = X[0].clone()
    Y, XH, YR = ctx.apply_A(X), ctx.apply_AH(y), ctx.residual(z, X)
    E1 = ctx.mec_cgls(y, 3, 1e-36)
    # frames in one chunk: the last ten, which the chunks split 8 + 2
    sub = slice(8, 18)
    c2 = ag.AltGDmin(512, 512, 8, 10, 1, int(cs.y.shape[2]), 1)
    c2.set_problem(torch.from_numpy(cs.coils.astype(np.complex64)).to(dev),
                   torch.from_numpy(np.ascontiguousarray(cs.mask[sub])).to(dev),
                   torch.from_numpy(np.ascontiguousarray(cs.m_k[sub])).to(dev), y[sub].contiguous())
    log("  operators")
    assert torch.equal(Y[sub], c2.apply_A(X[sub].contiguous()))
    assert torch.equal(XH[sub], c2.apply_AH(y[sub].contiguous()))
    assert torch.equal(YR[sub], c2.residual(z, X[sub].contiguous()))
    for k in (0, 15, 16, 17):  # MEC-1 frame by frame
        e, _ = R.cgls(lambda v: cs.op.A(k, v), lambda w: cs.op.AH(k, w), cs.y[k, :, : cs.m_k[k]],
                      np.zeros(p.n, dtype=np.complex128), 1e-36, 3)
        d = rel(E1[k].cpu().numpy().astype(np.complex128), e)
        log(f"  MEC-1 frame {k}: {d:.1e}")
        assert d < 5e-5
    ref = R.mec2(cs.op, cs.y, max_iter=2, tol=0.0)
    E2, it = ctx.mec_ista(y, 2, 1e-3, 0.0, sync=True)
    d = rel(E2.cpu().numpy().astype(np.complex128).T, ref.E)
    log(f"  MEC-2 after {it} updates: {d:.1e}")
    assert it == 2 and d < 5e-5
