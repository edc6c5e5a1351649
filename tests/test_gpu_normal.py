"""The fused normal operator behind the mean image and MEC-1, through the C
ABI against the FP64 oracle, over every transform length of its tiles (8 to
512, either axis), images narrower than a column tile, one and several coil
groups, both mask kinds and frames of unequal length.

Tolerance: a transform pair of length N rounds by about log2(N) * 2^-24
relative (under 6e-7 at N = 512 for both axes), and one CG iteration can
carry a rounding error forward by the ratio of successive residuals (below
4 here): three iterations stay under 6e-7 * 4^3 = 4e-5; 5e-5 is asserted."""
import numpy as np
import pytest

import datagen
from oracle import mri as R

from gpu_cases import GPU_OK, Case, log, rel

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch

SHAPES = [  # nx, ny, nc, q, kind, lines or samples
    (8, 8, 1, 2, "lines", 3), (8, 8, 2, 3, "index", 20), (16, 512, 3, 2, "lines", 100), (512, 16, 2, 2, "index", 2000),
    (16, 512, 2, 2, "index", 2000), (64, 256, 7, 3, "lines", 40), (256, 64, 5, 2, "index", 3000),
    (128, 32, 13, 9, "lines", 9), (32, 128, 4, 33, "index", 700), (512, 128, 2, 2, "lines", 30),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}c{s[2]}q{s[3]}{s[4]}")
def test_mean_and_mec1_over_tile_shapes(shape):
    nx, ny, nc, q, kind, lm = shape
    p = datagen.make_small(nx, ny, nc, q, 1, seed=11, kind=kind, n_lines=lm, m=lm, lowrank=False, snr_db=30.0,
                           variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx()
    z, it = ctx.mean(1e-3, 3, sync=True)
    zr, itr = R.mean_image(cs.op, cs.y, tol=1e-3, maxit=3)
    E = ctx.mec_cgls(torch.from_numpy(cs.y32).cuda(), 3, 1e-36)
    Er = R.mec1(cs.op, cs.y)
    ez = rel(z.cpu().numpy().astype(np.complex128), zr)
    ee = rel(E.cpu().numpy().astype(np.complex128).T, Er)
    log(f"  {shape}: mean rel {ez:.2e}, MEC-1 rel {ee:.2e}")
    assert it == itr and ez < 5e-5 and ee < 5e-5
    z0, it0 = ctx.mean(0.0, 0, sync=True)  # no iteration: the zero image
    assert it0 == 0 and not z0.any() and not ctx.mec_cgls(torch.from_numpy(cs.y32).cuda(), 0, 0.0).any()


@pytest.mark.parametrize("q,kind", [(1, "lines"), (2, "index"), (3, "lines"), (31, "lines"), (32, "index"), (62, "lines"),
                                    (64, "index"), (95, "lines"), (127, "index"), (128, "lines")])
def test_mec2_over_frame_counts(q, kind):
    """ISTA's temporal step at the edges of its tiles of 16 frequencies (0 to
    q/2), odd and even frame counts.  Every update's map is nonexpansive, so
    the rounding of ten updates adds up: two DFTs over q frames (half-length
    sums, below 1e-6 each) and the operator's four transforms (below 1e-6)
    per update, 3e-5 in all; 5e-5 is asserted."""
    p = datagen.make_small(16, 8, 2, q, 1, seed=13, kind=kind, n_lines=4, m=50, lowrank=False, snr_db=30.0,
                           variable_m=True)
    cs = Case(p)
    ctx = cs.gpu_ctx()
    ref = R.mec2(cs.op, cs.y, tol=0.0)
    E, it = ctx.mec_ista(torch.from_numpy(cs.y32).cuda(), 10, 1e-3, 0.0, sync=True)
    e = rel(E.cpu().numpy().astype(np.complex128).T, ref.E)
    log(f"  q {q} {kind}: updates gpu {it} oracle {ref.iters}; rel {e:.2e}")
    assert it == ref.iters and e < 5e-5
    E, it = ctx.mec_ista(torch.from_numpy(cs.y32).cuda(), 0, 1e-3, 0.0, sync=True)  # no update: zero
    assert it == 0 and not E.any()
