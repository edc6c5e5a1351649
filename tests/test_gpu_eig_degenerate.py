"""The spectral initialisation's eigenproblem on degenerate sequences, through
the spectrum it reports and the basis it gives: identical frames, exact low
rank, orthogonal frames of equal and of graded energy, frames that are zero,
repeated or far apart in scale, and sequences of very small and very large
values.  One coil of ones and every line sampled make X_0 the sequence itself
(scaled), so that the reference is the sequence's own FP64 SVD.

Tolerance: X_0 carries the FP32 rounding of two transforms of length 16 (each
below 16 roundings, 2^-20 relative), so a squared singular value moves by at most
2 * 2^-20 sigma_1^2 = 2e-6 sigma_1^2, and the projector of the leading r by
2 * 2^-20 sigma_1 / gap; both are asserted, the latter where the gap carries it."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, log, proj_dist

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch
    import paper_2212_09664_amd as ag

N = 256


def _sequence(kind, q, rng):
    """n x q, and the rank that its energy carries."""
    if kind == "identical":
        return np.repeat(datagen.crandn(rng, N, 1), q, axis=1), 1
    if kind == "proportional":  # one image, frames 1e-3 to 1e3 of it
        return datagen.crandn(rng, N, 1) * np.logspace(-3, 3, q)[None, :], 1
    if kind == "rank3":
        return datagen.crandn(rng, N, 3) @ datagen.crandn(rng, 3, q), min(3, q)
    if kind == "pairs":  # every frame twice
        return np.repeat(datagen.crandn(rng, N, (q + 1) // 2), 2, axis=1)[:, :q], min(16, (q + 1) // 2)
    if kind == "one_frame":  # all but one are zero
        Z = np.zeros((N, q), complex)
        Z[:, q // 2] = datagen.crandn(rng, N)
        return Z, 1
    if kind == "orthogonal":  # one pixel each: the Gram is a multiple of the identity
        return 3.0 * np.eye(N, q).astype(complex), min(16, q)
    if kind == "graded":
        return np.eye(N, q) * np.logspace(0, -1, q)[None, :] + 0j, min(5, q)
    return datagen.crandn(rng, N, q), min(16, q)


@pytest.mark.parametrize("q", [2, 3, 8, 17, 40, 64, 65, 100, 128])
@pytest.mark.parametrize("kind", ["identical", "proportional", "rank3", "pairs", "one_frame", "orthogonal", "graded",
                                  "random"])
def test_spectrum_and_basis(kind, q):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(q)
    Z0, r = _sequence(kind, q, rng)
    for scale in (1.0, 1e-12, 1e12):
        Z = (scale * Z0).astype(np.complex64)
        y = np.fft.fft2(Z.astype(np.complex128).T.reshape(q, 16, 16), norm="ortho").astype(np.complex64)
        ctx = ag.AltGDmin(16, 16, 1, q, r, N, trunc_c=0.0)
        ctx.set_problem(torch.ones(1, N, dtype=torch.complex64, device=dev),
                        torch.arange(16, dtype=torch.int32, device=dev).repeat(q, 1),
                        torch.full((q,), N, dtype=torch.int32, device=dev),
                        torch.from_numpy(y.reshape(q, 1, N)).to(dev))
        cap = min(16, q)
        e = np.array(ctx.rank_energy(cap))
        u, s, _ = np.linalg.svd(Z.astype(np.complex128), full_matrices=False)
        ref = s[:cap] ** 2 / N ** 2  # X_0 = A^H y / sqrt(m_k mbar), m_k = mbar = n
        err = np.max(np.abs(e - ref)) / ref[0]
        gap = (s[r - 1] - (s[r] if r < len(s) else 0.0)) / s[0]
        d = None
        if gap > 1e-3:
            U = ctx.init().cpu().numpy().astype(np.complex128).T
            assert ctx.last_error()[0] == 0
            d = proj_dist(U, u[:, :r])
        log(f"  {kind}, q {q}, scale {scale:.0e}: spectrum {err:.1e}, rank {r}, gap {gap:.1e}, projector {d}")
        assert np.all(np.isfinite(e)) and err < 2e-6
        assert d is None or d < np.sqrt(2 * r) * 2.0 ** -19 / gap
