"""The step's rules above rank 8 (each class of its register rows): the exit
rule against the oracle, the two ways its outcome is committed against each
other, the cap on the step size, and a step whose Gram partials are too many to
be summed inside it (more than 96 KB: a launch of their own sums them).

Tolerances: those of test_gpu_parity's tests of the same rules up to rank 8, and
of test_gpu_step's step; the partials are FP32 sums over at most 256 pixels
(an image column or a block of rows), below 256 * 2^-24 = 1.5e-5."""
import numpy as np
import pytest

import datagen
from oracle import altgdmin as AG

from gpu_cases import GPU_OK, Case, from_gpu_B, from_gpu_U, log, rel, to_gpu_U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


def _case(r, q):
    return Case(datagen.make_small(32, 32, 6, q, r, seed=43, kind="lines", n_lines=16, lowrank=True, snr_db=40.0,
                                   variable_m=True))


@pytest.mark.parametrize("r,q", [(9, 40), (12, 48), (13, 52), (16, 64)])
def test_exit_rule(r, q):
    eps = 0.01
    cs = _case(r, q)
    ref = AG.run(cs.op, cs.y, AG.Params(r=r, eps_exit=eps), record=True)
    sd = np.array(ref.history["sd"]) / np.sqrt(r)
    assert ref.history["exit_at"] == ref.iters and ref.iters < 70
    assert np.min(np.abs(sd - eps)) > 0.01 * eps
    ctx = cs.gpu_ctx(eps_exit=eps)
    U = ctx.init()
    Uprev = torch.empty_like(U)
    B, done = ctx.iterate(70, U, U_prev=Uprev, sync=True)
    st = ctx.stats()
    e = rel(from_gpu_U(Uprev) @ from_gpu_B(B), ref.X)
    log(f"  r {r}: iterations gpu {done} oracle {ref.iters}; X {e:.1e}; sd/sqrt(r) {st['sd'] / np.sqrt(r):.6f}")
    assert done == ref.iters and st["t"] == ref.iters and st["exited"] == 1
    assert st["sd"] / np.sqrt(r) == pytest.approx(sd[-1], rel=1e-3) and e < 1e-3


@pytest.mark.parametrize("r,q", [(9, 40), (12, 48), (13, 52), (16, 64)])
def test_commit_paths_agree(r, q):
    """A threshold that never fires leaves the trajectory bitwise unchanged."""
    cs = _case(r, q)
    out = []
    for eps in (0.0, 1e-30):
        ctx = cs.gpu_ctx(eps_exit=eps)
        U = ctx.init()
        B, done = ctx.iterate(10, U, sync=True)
        out.append((U.clone(), B.clone(), done, ctx.get_eta(), ctx.stats()))
    (Ua, Ba, da, ea, sa), (Ub, Bb, db, eb, sb) = out
    assert da == db == 10 and sa["t"] == sb["t"] == 10 and sa["exited"] == sb["exited"] == 0
    assert torch.equal(Ua, Ub) and torch.equal(Ba, Bb)
    assert ea == eb and sa["f"] == sb["f"] and sa["sd"] == sb["sd"]


@pytest.mark.parametrize("r,q", [(9, 40), (13, 52)])
@pytest.mark.parametrize("bind", [True, False], ids=["cap_binds", "cap_loose"])
def test_step_size_cap(bind, r, q):
    cs = _case(r, q)
    T = 6
    free = AG.run(cs.op, cs.y, AG.Params(r=r), t_fixed=1, record=False)
    cap1 = AG.step_size_cap(cs.op, AG.ls_step(cs.op, free.U0, cs.y), 1.0)
    c = (0.5 if bind else 2.0) * free.eta / cap1
    ref = AG.run(cs.op, cs.y, AG.Params(r=r, eta_cap_c=c), t_fixed=T, record=True)
    assert ref.history["eta_capped"] is bind
    ctx = cs.gpu_ctx(eta_cap_c=c)
    U = ctx.init()
    Uprev = torch.empty_like(U)
    B, done = ctx.iterate(T, U, U_prev=Uprev, sync=True)
    e = rel(from_gpu_U(Uprev) @ from_gpu_B(B), ref.X)
    log(f"  r {r}, binds {bind}: eta gpu {ctx.get_eta():.6e} oracle {ref.eta:.6e}; X {e:.1e}")
    assert done == T and ctx.get_eta() == pytest.approx(ref.eta, rel=1e-4) and e < 1e-3


def _qr(A):
    Q, R = np.linalg.qr(A)
    return Q * (np.diag(R) / np.abs(np.diag(R)))[None, :]


@pytest.mark.parametrize("nx,ny,r,precision,kib", [(256, 64, 4, 0, 72), (256, 64, 5, 0, 110), (128, 64, 9, 0, 171),
                                                   (128, 64, 12, 1, 150), (64, 128, 16, 0, 264), (64, 128, 16, 1, 264)])
def test_step_from_many_partials(nx, ny, r, precision, kib):
    """kib: the partials (2r columns' triangle per image column, 8 bytes an
    entry, or per 256 pixels, 16 bytes in the mixed form), on either side of 96."""
    n = nx * ny
    assert (nx * 8 if precision == 0 else n // 256 * 16) * r * (2 * r + 1) // 1024 == kib
    p = datagen.make_small(nx, ny, 4, 24, r, seed=60 + r, kind="lines", n_lines=ny // 3, lowrank=True, snr_db=20.0,
                           variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx(precision=precision)
    U0 = _qr(datagen.crandn(np.random.default_rng(r), n, r)).astype(np.complex64)
    U = ctx.init_from(to_gpu_U(U0))
    U0 = from_gpu_U(U)
    Gn = from_gpu_U(ctx.gradient(U)[1])
    ctx.iterate(1, U)
    st = ctx.stats()
    eta = 0.14 / np.linalg.norm(Gn, 2)
    e1, ee = rel(from_gpu_U(U), _qr(U0 - eta * Gn)), abs(st["eta"] / eta - 1)
    eg = abs(st["grad_norm"] / np.linalg.norm(Gn) - 1)
    log(f"  {nx} x {ny}, r {r}, precision {precision}, {kib} KiB: step {e1:.1e}, eta {ee:.1e}, grad {eg:.1e}")
    assert e1 < 5e-5 and ee < 5e-5 and eg < 5e-5
