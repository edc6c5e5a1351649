"""The statistics of the last iteration where a captured LS step, recorded
before the context's first iteration, is replayed after it: the solve
overwrites the frames' costs, and what get_stats reports is still the
iteration's (ranks on either side of 8, 128 frames at the limit)."""
import numpy as np
import pytest

import datagen

from gpu_cases import GPU_OK, Case, log, to_gpu_U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not GPU_OK, reason="needs a GPU")]

if GPU_OK:
    import torch
    import paper_2212_09664_amd as ag


@pytest.mark.parametrize("q,r", [(12, 4), (40, 11), (128, 9)])
def test_statistics_survive_a_replayed_ls_step(q, r):
    p = datagen.make_small(32, 32, 3, q, r, seed=52, kind="lines", n_lines=14, lowrank=True, snr_db=40.0)
    cs = Case(p)
    other = to_gpu_U(np.linalg.qr(datagen.crandn(np.random.default_rng(3), p.n, r))[0])
    dev, s = torch.device("cuda:0"), torch.cuda.Stream()
    want = None
    for eps, replay in ((1e-30, False), (0.0, False), (0.0, True)):  # statistics formed at once, then deferred
        ctx = ag.AltGDmin(p.nx, p.ny, p.nc, q, r, int(cs.y.shape[2]), eps_exit=eps)
        with torch.cuda.stream(s):
            ctx.set_problem(torch.from_numpy(cs.coils.astype(np.complex64)).to(dev), torch.from_numpy(cs.mask).to(dev),
                            torch.from_numpy(cs.m_k).to(dev), torch.from_numpy(cs.y32).to(dev), stream=s)
            U, B = ctx.init(), torch.empty(q, r, dtype=torch.complex64, device=dev)
        s.synchronize()
        if replay:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                ctx.ls(other, B)
        with torch.cuda.stream(s):
            for _ in range(2):  # two rounds of iterations, each followed by a replay
                ctx.iterate(3, U)
                if replay:
                    g.replay()
        st = ctx.stats()
        want = want or st
        log(f"  q {q} r {r} replay {replay}: f {st['f']:.9e} of {want['f']:.9e}, t {st['t']}")
        assert st["t"] == 6
        assert st["f"] == pytest.approx(want["f"], rel=1e-12)
        assert st["sd"] == pytest.approx(want["sd"], rel=1e-9)
        assert st["grad_norm"] == pytest.approx(want["grad_norm"], rel=1e-12)
