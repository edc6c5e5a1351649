"""The spectral initialisation's q x q eigenproblem at the edges of its layout:
one register row per lane up to 64 frames and two above, eight waves' columns
(frame counts around multiples of 8), one or two eigenvectors per wave (rank 8
and 9), the inverse iteration's room in LDS (rank 16 around 122 frames), and the
smallest frame counts.  Against the oracle's spectral initialisation.

Tolerance: the basis is X_0 V / Sigma in FP32 from an FP64 eigenproblem whose
matrix carries X_0's FP32 rounding; the projector's error is below 1e-6 over the
relative gap at the rank, the bound the other initialisation tests use."""
import numpy as np
import pytest

import datagen

from oracle import altgdmin as AG
from gpu_cases import GPU_OK, Case, from_gpu_U, log, proj_dist

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]


@pytest.mark.parametrize("q,r", [(1, 1), (2, 1), (2, 2), (3, 2), (7, 3), (8, 2), (9, 3), (17, 5), (33, 8), (63, 9),
                                 (64, 16), (65, 16), (72, 8), (97, 9), (113, 12), (121, 16), (122, 16), (123, 16),
                                 (127, 11), (128, 8)])
def test_eigenvectors(q, r):
    p = datagen.make_small(32, 16, 3, q, r, seed=100 + q, kind="lines", n_lines=9, lowrank=True, snr_db=40.0)
    cs = Case(p)
    U0 = from_gpu_U(cs.gpu_ctx().init())
    Ytr, _, _ = AG.truncation(cs.op, cs.y, 36.0)
    X0 = AG.backprojection(cs.op, Ytr)
    s = np.append(np.linalg.svd(X0, compute_uv=False), 0.0)
    gap = (s[r - 1] - s[r]) / s[0]
    d = proj_dist(U0, AG.spectral_init(X0, r))
    log(f"  q {q} r {r}: projector distance {d:.2e}, relative gap {gap:.2e}")
    assert np.allclose(U0.conj().T @ U0, np.eye(r), atol=2e-6)
    assert d < 1e-6 / gap
