"""Short STGD runs at the edges of the column kernel's tiles, against the FP64
oracle on identical inputs: k on both sides of every tile count (and k + 1, k + 2
at a tile's end, where the folded means fit or do not), batches that end inside
a chunk of 16 or 32 rows, a ragged last batch, one view and three, a run that is
shorter than the staging depth and one that is longer.

Bars: the summed update Phi_T - Phi_0 matches the oracle's within 1e-5 relative
(FP32, the bar of a single step: each step's update is right to 1e-5 and the
updates add up with the same sign pattern) and 3e-2 (BF16 operands: 2^-8 for
each of the three operands that a direction passes through)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import bf16_round, dev, f32_round, padded, phi_cols, phi_rows, rel, to_dev

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 14, 15, 16, 17, 30, 33, 48, 63, 65, 80, 94, 97, 112, 113, 128])
@pytest.mark.parametrize("three", [False, True])
@pytest.mark.parametrize("dtype,batch,tail,compensated",
                         [("fp32", 16, 0, True), ("fp32", 33, 5, False), ("fp32", 128, 100, True),
                          ("bf16", 17, 3, True), ("bf16", 48, 47, False), ("bf16", 100, 33, False), ("bf16", 128, 1, True)])
@pytest.mark.parametrize("steps", [1, 5])
def test_short_run(k, three, dtype, batch, tail, compensated, steps):
    n = (steps - 1) * batch + (tail or batch)
    g = np.random.default_rng(1000 * k + batch + steps)
    lo = bf16_round if dtype == "bf16" else f32_round
    views = [lo(g.standard_normal((n, k)) * 0.3 + s) for s in ((0.2, 0.1, -0.1) if three else (0.2,))]
    views = views if three else views * 3
    ybar = f32_round(np.stack([v.mean(0) for v in views]))
    Phi0 = f32_round(synth.initial_factors(k, seed=k) * 1.1)
    perm = g.permutation(n).astype(np.int32)
    beta0, tau, alpha0 = 0.01, 50.0, 0.5
    ref = Phi0
    for t in range(steps):
        rows = perm[t * batch:(t + 1) * batch]
        ref = oracle.sgd_step(views[0][rows], views[1][rows], views[2][rows], ybar, ref, beta0 / (1 + t / tau), alpha0)
    ldy, tdt = otm.default_ldy(k), torch.bfloat16 if dtype == "bf16" else torch.float32
    Y = [padded(v, ldy, tdt) for v in (views if three else views[:1])]
    Y = Y if three else Y * 3
    P = phi_rows(Phi0)
    p = otm.SgdParams(k=k, batch=batch, passes=1, alpha0=alpha0, beta0=beta0, beta_tau=tau, compensated=compensated,
                      y_dtype=otm.BF16 if dtype == "bf16" else otm.F32)
    otm.sgd_run(p, n, *Y, to_dev(ybar), torch.from_numpy(perm)[None].contiguous().to(dev()), P)
    torch.cuda.synchronize()
    assert rel(phi_cols(P) - Phi0, ref - Phi0) < (3e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("k,three,compensated,batch",
                         [(k, True, False, b) for k in (65, 78, 79, 95, 96) for b in (112, 113, 128)]
                         + [(k, False, True, b) for k in (112, 113, 120, 126, 127) for b in (89, 90, 128)]
                         + [(k, three, c, b) for k in (1, 10, 14, 16, 17, 30) for three in (False, True)
                            for c, b in ((False, 48), (False, 49), (True, 64), (True, 65))])
@pytest.mark.parametrize("steps", [1, 4])
def test_rules_between_the_kernels(k, three, compensated, batch, steps):
    """Both sides of the rules that send BF16 runs to the grid
    kernel, with a ragged last batch (and the k whose last tile holds only padding)."""
    test_short_run(k, three, "bf16", batch, batch - 29, compensated, steps)


@pytest.mark.parametrize("k,three,batch", [(16, False, 32), (17, False, 33), (31, False, 100), (46, False, 17), (47, False, 48),
                                           (47, False, 49), (49, False, 16), (62, False, 100), (63, False, 49), (64, False, 128), (65, False, 48),
                                           (3, True, 17), (14, True, 48), (16, True, 100), (32, True, 33), (33, True, 48)])
@pytest.mark.parametrize("compensated", [False, True])
@pytest.mark.parametrize("restarts", [256, 257])
def test_more_restarts_than_cus(k, three, batch, compensated, restarts):
    """Both sides of the rule for many restarts: two workgroups to a CU.  Every restart
    has the same start and rows, so all end with the same bits; they match the oracle."""
    steps, tail = 3, batch // 2 + 1
    n = (steps - 1) * batch + tail
    g = np.random.default_rng(1000 * k + batch)
    views = [bf16_round(g.standard_normal((n, k)) * 0.3 + s) for s in ((0.2, 0.1, -0.1) if three else (0.2,))]
    views = views if three else views * 3
    ybar = f32_round(np.stack([v.mean(0) for v in views]))
    Phi0 = f32_round(synth.initial_factors(k, seed=k) * 1.1)
    ref = Phi0
    for t in range(steps):
        rows = slice(t * batch, (t + 1) * batch)
        ref = oracle.sgd_step(views[0][rows], views[1][rows], views[2][rows], ybar, ref, 0.01 / (1 + t / 50.0), 0.5)
    Y = [padded(v, otm.default_ldy(k), torch.bfloat16) for v in (views if three else views[:1])]
    P = phi_rows(Phi0).repeat(restarts, 1, 1).contiguous()
    p = otm.SgdParams(k=k, batch=batch, passes=1, alpha0=0.5, beta0=0.01, beta_tau=50.0, compensated=compensated,
                      y_dtype=otm.BF16)
    otm.sgd_run(p, n, *(Y if three else Y * 3), to_dev(ybar), None, P, restarts=restarts)
    torch.cuda.synchronize()
    assert torch.equal(P, P[:1].expand_as(P))
    assert rel(phi_cols(P[0]) - Phi0, ref - Phi0) < 3e-2
