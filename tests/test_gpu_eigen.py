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


@pytest.mark.parametrize("kt", [66, 100, 200])
@pytest.mark.parametrize("kind", ["low rank", "three", "equal", "pairs", "clump", "identity"])
def test_equal_eigenvalues_take_no_rotations(kt, kind):
    """Eigenvalues equal to rounding errors are no reason to run the rotations after the
    direct solver: their log, the largest part of the workspace, stays as it was.  Both
    eigenproblems of the call (kt columns each, past 64) are the direct solver's."""
    g = np.random.default_rng(kt)
    lam = {"low rank": np.where(np.arange(kt) < kt // 2, np.linspace(9.0, 1.0, kt), 0.0),
           "three": np.where(np.arange(kt) < 3, 3.0 - np.arange(kt), 0.0),
           "equal": np.repeat([4.0, 1.0], [kt // 2, kt - kt // 2]),
           "pairs": np.repeat(np.linspace(1.0, 9.0, kt // 2), 2),
           "clump": np.where(np.arange(kt) < kt // 2, 3.0, np.linspace(1.0, 9.0, kt)),
           "identity": np.ones(kt)}[kind]
    V = np.linalg.qr(g.standard_normal((kt, kt)))[0]
    M = (V * lam) @ V.T
    M = 0.5 * (M + M.T)
    S = np.linalg.qr(g.standard_normal((3 * kt, kt)))[0]
    O, St = to_dev(S @ M, torch.float64), to_dev(S, torch.float64)
    ws = torch.full((otm.lib().otm_whitener_workspace(3 * kt, kt, kt),), 0xA5, dtype=torch.uint8, device=dev())
    W = torch.empty((3 * kt, kt), dtype=torch.float64, device=dev())
    ev = torch.empty(kt, dtype=torch.float64, device=dev())
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm._check(otm.lib().otm_whitener(O.data_ptr(), St.data_ptr(), 3 * kt, kt, kt, W.data_ptr(), ev.data_ptr(), None,
                                      otm.F32, kt, info.data_ptr(), ws.data_ptr(), ws.numel(), otm._stream()))
    assert int(info.item()) == (1 if lam.min() == 0.0 else 0)
    log_bytes = 60 * (kt - 1) * (kt // 2) * 20               # 60 sweeps of 16-byte rotations and 4-byte pairs
    untouched = int((ws == 0xA5).sum().item())
    assert untouched >= log_bytes
    if lam.min() > 0.0:
        P = S.T @ W.cpu().numpy()
        assert np.abs(P.T @ M @ P - np.eye(kt)).max() < 4 * kt * 2.0**-52 * lam.max() / lam.min()
        assert np.abs(ev.cpu().numpy() - np.sort(lam)[::-1]).max() < 1e-12 * lam.max()


@pytest.mark.parametrize("k", [33, 64, 65, 100, 128])
def test_unwhitening_takes_rotations(k):
    """The Gram of a whitener's columns is diagonal to rounding, one sweep of the
    rotations: their log is written, and nothing of the direct solver's part of the workspace
    (more than six k x k matrices) beside it."""
    g = np.random.default_rng(k)
    W = np.linalg.qr(g.standard_normal((300, k)))[0] * np.linspace(1.0, 9.0, k)
    Wt, Phi = to_dev(W, torch.float64), torch.eye(k, device=dev())
    ws = torch.full((otm.lib().otm_unwhiten_workspace(300, k),), 0xA5, dtype=torch.uint8, device=dev())
    mu = torch.empty((300, k), dtype=torch.float64, device=dev())
    ah, lam = (torch.empty(k, dtype=torch.float64, device=dev()) for _ in range(2))
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm._check(otm.lib().otm_unwhiten_topics(Wt.data_ptr(), 300, k, Phi.data_ptr(), 1.0, mu.data_ptr(), ah.data_ptr(),
                                             lam.data_ptr(), info.data_ptr(), ws.data_ptr(), ws.numel(), otm._stream()))
    assert int(info.item()) == 0
    players = (k + 1) // 2 * 2
    sweep = (players - 1) * (players // 2)
    written = int((ws != 0xA5).sum().item())
    # the call's own five matrices and column sums, one sweep of 20-byte rotations
    assert written <= 8 * (5 * k * k + 131 * k) + 20 * sweep + 4096
    ref = W @ np.linalg.inv(W.T @ W)
    ref = np.maximum(ref, 0.0)
    assert np.abs(mu.cpu().numpy() - ref / ref.sum(0)).max() < 1e-12
