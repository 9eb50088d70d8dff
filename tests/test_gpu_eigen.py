"""The eigensolver behind the whitener at the sizes where its path changes (32 and
33, 64 and 65, the 64-column blocks, 200 and 201) and on spectra that its direct form must hand
to the rotations (equal and nearly equal eigenvalues) or meets as they are (blocks
that do not couple, a diagonal matrix): Omega = S^T O with S orthonormal and O = S M,
M symmetric positive definite of kt x kt, so the whitener's eigenvalues are M's.

Bars: eigenvalues within 1e-12 of the largest (working precision times the size),
W^T (S M S^T) W = I within 1e-9, the whitener's own bar for well-conditioned M."""
import numpy as np
import pytest
import torch

from gpu_util import dev, to_dev

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


def _matrix(kt, kind, g):
    V = np.linalg.qr(g.standard_normal((kt, kt)))[0]
    if kind == "spread":
        lam = np.linspace(1.0, 50.0, kt) * (1 + 0.2 * g.random(kt))
    elif kind == "close":
        lam = 1.0 + np.sort(g.random(kt)) * 1e-7
        lam[: kt // 2] += 3.0
    elif kind == "equal":
        lam = np.repeat([4.0, 1.0], [kt // 2, kt - kt // 2])
    elif kind == "diagonal":
        return np.diag(np.linspace(1.0, 9.0, kt)[g.permutation(kt)])
    else:                                   # two blocks that do not couple
        lam = np.linspace(1.0, 20.0, kt)
        h = kt // 3
        V = np.zeros((kt, kt))
        V[:h, :h] = np.linalg.qr(g.standard_normal((h, h)))[0]
        V[h:, h:] = np.linalg.qr(g.standard_normal((kt - h, kt - h)))[0]
    M = (V * lam) @ V.T
    return 0.5 * (M + M.T)


@pytest.mark.parametrize("kt", [20, 32, 33, 48, 64, 65, 100, 128, 129, 192, 193, 200, 201])
@pytest.mark.parametrize("kind", ["spread", "close", "equal", "diagonal", "blocks"])
def test_whitener_spectra(kt, kind):
    g = np.random.default_rng(kt)
    d = 3 * kt + 1
    S = np.linalg.qr(g.standard_normal((d, kt)))[0]
    M = _matrix(kt, kind, g)
    W, ev, _ = otm.whitener(to_dev(S @ M, torch.float64), to_dev(S, torch.float64), kt, w_lo_dtype=None)
    W, ev = W.cpu().numpy(), ev.cpu().numpy()
    ref = np.linalg.eigvalsh(M)[::-1]
    assert np.abs(ev - ref).max() < 1e-12 * ref[0]
    P = S.T @ W
    assert np.abs(P.T @ M @ P - np.eye(kt)).max() < 1e-9


@pytest.mark.parametrize("kt", [33, 64, 65, 100, 200])
@pytest.mark.parametrize("gap", [1e-4, 1e-5, 1e-6, 2e-7, 1e-8])
def test_close_eigenvalues_keep_the_precision(kt, gap):
    """Eigenvectors stay orthogonal to working precision whatever the gaps, so W whitens
    to it.  Bar: four times n 2^-52, the rounding errors of sums of n terms (the
    eigenvalues lie within 2% of one another, so nothing enlarges them)."""
    g = np.random.default_rng(kt)
    S = np.linalg.qr(g.standard_normal((3 * kt, kt)))[0]
    V = np.linalg.qr(g.standard_normal((kt, kt)))[0]
    M = (V * (1.0 + gap * np.arange(kt))) @ V.T
    M = 0.5 * (M + M.T)
    W, _, _ = otm.whitener(to_dev(S @ M, torch.float64), to_dev(S, torch.float64), kt, w_lo_dtype=None)
    P = S.T @ W.cpu().numpy()
    assert np.abs(P.T @ M @ P - np.eye(kt)).max() < 4 * kt * 2.0**-52
