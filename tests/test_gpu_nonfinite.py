"""NaN and infinite inputs of the FP64 stages: every call returns, says so where it has a
status, and what does not depend on the bad entry is right.

Sizes on both sides of every solver of the eigenproblems (32 and 33, 64 and 65, 200
and 201) and of the orthonormalization (200 and 201)."""
import numpy as np
import pytest
import torch

from gpu_util import dev, to_dev

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf"), float("-inf")]


@pytest.mark.parametrize("kt", [20, 32, 33, 64, 65, 200, 201])
@pytest.mark.parametrize("bad", BAD)
def test_whitener_refuses(kt, bad):
    """The list of eigenvalues by size is whole whatever they are (its entries are read
    as column numbers).  NaN is reported; -inf may pass for the smallest eigenvalue, and
    then the columns show it."""
    g = np.random.default_rng(kt)
    d, k = 2 * kt, kt // 2
    S = np.linalg.qr(g.standard_normal((d, kt)))[0]
    O = S * np.linspace(2.0, 1.0, kt)
    O[3, 5] = bad
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    W, ev, _ = otm.whitener(to_dev(O, torch.float64), to_dev(S, torch.float64), k, w_lo_dtype=None, info=info)
    assert int(info.item()) == 1 or (np.isinf(bad) and not torch.isfinite(W).all())


@pytest.mark.parametrize("m", [20, 64, 200, 201])
@pytest.mark.parametrize("bad", BAD)
def test_orthonormalize_refuses(m, bad):
    g = np.random.default_rng(m)
    Y = g.standard_normal((2 * m + 1, m))
    Y[4, m - 1] = bad
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm.orthonormalize(to_dev(Y, torch.float64), info=info)
    assert int(info.item()) == 1


@pytest.mark.parametrize("k", [20, 33, 65, 128])
@pytest.mark.parametrize("bad", BAD)
def test_unwhiten_refuses(k, bad):
    g = np.random.default_rng(k)
    W = g.standard_normal((4 * k, k))
    W[7, 2] = bad
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm.unwhiten_topics(to_dev(W, torch.float64), torch.eye(k, device=dev()), info=info)
    assert int(info.item()) == 1


@pytest.mark.parametrize("m,k", [(20, 10), (65, 33), (200, 100), (201, 100)])
@pytest.mark.parametrize("bad", BAD)
def test_pinv_factors_refuse(m, k, bad):
    g = np.random.default_rng(m)
    J, K, S = (g.standard_normal((3 * m, m)) for _ in range(3))
    J[1, 4] = bad
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm.pinv_factors(*(to_dev(x, torch.float64) for x in (J, K, S)), k, info=info)
    assert int(info.item()) != 0


@pytest.mark.parametrize("k", [1, 16, 17, 100, 128])
@pytest.mark.parametrize("bad", BAD)
def test_recover_pi_keeps_samples_apart(k, bad):
    """A bad entry of a sample reaches that sample's memberships only, and a sample
    whose products have no positive finite sum gets zeros."""
    g = torch.Generator().manual_seed(k)
    Y = torch.zeros((70, otm.default_ldy(k)))
    Y[:, :k] = torch.rand((70, k), generator=g) + 0.1
    clean = otm.recover_pi(Y.to(dev()), k, torch.eye(k, device=dev()), tau=0.0).cpu()
    Y[33, 0] = bad
    Pi = otm.recover_pi(Y.to(dev()), k, torch.eye(k, device=dev()), tau=0.0).cpu()
    keep = torch.arange(70) != 33
    assert torch.equal(Pi[:, keep], clean[:, keep])
    assert not torch.isinf(Pi[:, 33]).any() and (Pi[:, 33] == 0).any()
