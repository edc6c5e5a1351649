"""The fused QR step at every class of its register rows (ranks 1 to 4, 5 to 8,
9 to 12, 13 to 16, odd and even), through the C ABI against FP64 numpy.

Tolerances: the factor is FP64 of an FP64 Gram, so the basis is exact to its
FP32 storage (2^-24) and one substitution of r FP32 terms: below r * 2^-22 =
4e-6 at rank 16 for a basis of condition below 10.  The step size, SD and
||grad|| come from the FP32 Gram of [U grad] (sums of n = 512 products on the
matrix cores, below 512 * 2^-24 = 3e-5 in the worst case of one-sided
rounding): 5e-5."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, from_gpu_U, log, rel, to_gpu_U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch


def _qr(A):
    Q, R = np.linalg.qr(A)
    return Q * (np.diag(R) / np.abs(np.diag(R)))[None, :]


@pytest.mark.parametrize("kind", ["lines", "index"])
@pytest.mark.parametrize("r", [1, 2, 4, 5, 8, 9, 12, 13, 16])
def test_basis_and_first_step(r, kind):
    p = datagen.make_small(32, 16, 4, 20, r, seed=60 + r, kind=kind, n_lines=9, m=280, lowrank=True, snr_db=20.0,
                           variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx()
    rng = np.random.default_rng(r)
    A = _qr(datagen.crandn(rng, p.n, r)) @ (np.eye(r) + 0.3 * datagen.crandn(rng, r, r) / np.sqrt(r))
    A32 = A.astype(np.complex64).astype(np.complex128)
    U = ctx.init_from(to_gpu_U(A32), torch.empty(r, p.n, dtype=torch.complex64, device="cuda:0"))
    U0 = from_gpu_U(U)
    e0 = rel(U0, _qr(A32))
    _, G = ctx.gradient(U)
    Gn = from_gpu_U(G)
    Up = torch.empty_like(U)
    ctx.iterate(1, U, U_prev=Up)
    st = ctx.stats()
    eta = 0.14 / np.linalg.norm(Gn, 2)
    U1 = _qr(U0 - eta * Gn)
    sd = np.linalg.norm(U1 - U0 @ (U0.conj().T @ U1))
    e1, ee = rel(from_gpu_U(U), U1), abs(st["eta"] / eta - 1)
    es, eg = abs(st["sd"] / sd - 1), abs(st["grad_norm"] / np.linalg.norm(Gn) - 1)
    log(f"  r {r} {kind}: basis {e0:.1e}, step {e1:.1e}, eta {ee:.1e}, grad {eg:.1e}; SD {st['sd']:.4e} ({es:.1e})")
    assert torch.equal(Up.cpu(), torch.from_numpy(np.ascontiguousarray(U0.T.astype(np.complex64))))
    assert e0 < 4e-6 and e1 < 5e-5 and ee < 5e-5 and eg < 5e-5
    assert abs(st["sd"] ** 2 - sd ** 2) < 5e-5 * r  # SD^2 = r - ||U^H U+||^2
