"""The mean image's right-hand side A^H y is held in FP64 until the image is
rounded: after one iteration the image is a multiple of it, and its direction
is within one FP32 rounding of the 64-bit one, at every transform length.

Tolerance: a rounding to FP32 is 2^-24 / sqrt(3) rms at most.  Two act on the
direction (the right-hand side's and the update's: the step's own scale is
projected out), and on line masks the frames' FP32 row transforms, 2 log2(nx)
roundings whose mean over the f frames that sample a line is taken: for nx <= 32
and f >= 10 together below sqrt(2 + 10 / 10) 2^-24 / sqrt(3) = 2^-24.  (An FP32
adjoint of the frames' sum adds 2 log2(ny) of its own and the coils' sum.)"""
import numpy as np
import pytest

import datagen
from oracle import mri as R

from gpu_cases import GPU_OK, Case, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

SHAPES = [  # nx, ny, nc, q, kind, lines or samples
    (32, 128, 12, 40, "lines", 40), (8, 256, 16, 32, "lines", 128), (16, 512, 16, 24, "lines", 300),
    (16, 64, 9, 40, "lines", 20), (32, 32, 5, 30, "lines", 14), (32, 16, 3, 30, "lines", 8), (16, 8, 2, 30, "lines", 4),
    (64, 64, 8, 20, "index", 600), (128, 32, 7, 20, "index", 600), (256, 16, 4, 20, "index", 600),
    (512, 8, 4, 20, "index", 600), (8, 512, 4, 20, "index", 600), (16, 256, 1, 20, "index", 600),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}c{s[2]}q{s[3]}{s[4]}")
def test_right_hand_side_keeps_its_precision(shape):
    nx, ny, nc, q, kind, lm = shape
    p = datagen.make_small(nx, ny, nc, q, 2, seed=17, kind=kind, n_lines=lm, m=lm, lowrank=True, snr_db=30.0,
                           variable_m=True)
    p.zstar = p.zstar + 3 * np.abs(p.zstar).mean()  # a mean-dominated sequence
    cs = Case(p)
    z, it = cs.gpu_ctx().mean(0.0, 1, sync=True)
    z = z.cpu().numpy().astype(np.complex128)
    zr, _ = R.mean_image(cs.op, cs.y, tol=0.0, maxit=1)
    a = np.vdot(zr, z).real / np.vdot(zr, zr).real
    e = np.linalg.norm(z / a - zr) / np.linalg.norm(zr)
    log(f"  {shape}: direction {e:.2e} (scale off by {a - 1:.1e})")
    assert it == 1 and abs(a - 1) < 1e-5 and e < 2.0 ** -24
