"""Validation and membership recovery at the edges of their kernels: k_hat and k on
both sides of the 64 rows of a workgroup and the 4 of a thread, n around the 64
nodes of a staged chunk and the 384 of a split, more p-values than one 256-wide span
with ties among them; recovery with k around the 16-row tiles and n around 16 and 64
samples.

Bars: 1e-12 relative against float64 numpy (sums of at most 1000 terms), adjusted
p-values from the same p-values exactly as ranked; memberships within one float32
rounding (1e-6 relative) of the float64 expression."""
import numpy as np
import pytest
import torch

from gpu_util import dev, rel, to_dev

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kh,k", [(1, 1), (3, 5), (4, 64), (63, 65), (64, 64), (68, 129), (100, 100), (128, 128)])
@pytest.mark.parametrize("n", [3, 63, 64, 65, 383, 385, 1000])
def test_validate(kh, k, n):
    g = np.random.default_rng(kh * 1000 + k + n)
    A, B = g.random((kh, n)).astype(np.float32), g.random((k, n)).astype(np.float32)
    A[-1] = A[0]                                     # equal rows: equal p-values
    v = otm.validate(to_dev(A), to_dev(B), threshold=0.05)
    torch.cuda.synchronize()
    a, b = A.astype(np.float64), B.astype(np.float64)
    ac, bc = a - a.mean(1, keepdims=True), b - b.mean(1, keepdims=True)
    rho = ac @ bc.T / np.sqrt((ac**2).sum(1))[:, None] / np.sqrt((bc**2).sum(1))[None]
    assert np.abs(v.rho.cpu().numpy() - rho).max() < 1e-12
    l1 = np.stack([np.abs(a[i] - b).mean(1) for i in range(kh)])
    assert rel(v.l1.cpu().numpy(), l1) < 1e-12
    p = v.p.cpu().numpy().reshape(-1)
    m = p.size
    order = np.argsort(p, kind="stable")
    adj = np.empty(m)
    adj[order] = np.minimum(1.0, np.minimum.accumulate((p[order] * m / np.arange(1, m + 1))[::-1])[::-1])
    assert np.array_equal(v.p_adj.cpu().numpy().reshape(-1), adj)


@pytest.mark.parametrize("k", [1, 15, 16, 17, 33, 64, 100, 127, 128])
@pytest.mark.parametrize("n", [1, 15, 16, 63, 65, 200])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_recover_pi(k, n, dtype):
    g = torch.Generator().manual_seed(k + n)
    ldy = otm.default_ldy(k)
    Y = torch.zeros((n, ldy))
    Y[:, :k] = torch.randn((n, k), generator=g)
    Y = Y.to(dtype)
    Phi = torch.linalg.qr(torch.randn((k, k), generator=g))[0].contiguous() * 1.3
    Pi = otm.recover_pi(Y.to(dev()), k, Phi.to(dev()), tau=0.02).cpu().double().numpy()
    y, f = Y[:, :k].double().numpy(), Phi.double().numpy()
    nrm = np.sqrt((f**2).sum(1))
    x = np.maximum(f / nrm[:, None] / nrm[:, None] ** 3 @ y.T, 0)
    s = x.sum(0)
    x = np.where(s > 0, x / np.where(s > 0, s, 1), 0)
    near = np.abs(x - 0.02) < 1e-9                   # on the cut itself either side is right
    x[x < 0.02] = 0
    s = x.sum(0)
    x = np.where(s > 0, x / np.where(s > 0, s, 1), 0)
    assert np.abs(Pi - x)[:, ~near.any(0)].max(initial=0.0) < 1e-6


@pytest.mark.parametrize("k", [1, 2, 4, 8, 64])
def test_recover_pi_on_the_cut(k):
    """Entries that are exactly tau stay: k equal positive products have the quotient
    1 / k, exact in float64 for a k that is a power of two, whatever their size."""
    y = torch.arange(1, 200, dtype=torch.float32)
    Y = torch.zeros((y.numel(), otm.default_ldy(k)))
    Y[:, :k] = y[:, None]
    Pi = otm.recover_pi(Y.to(dev()), k, torch.eye(k, device=dev()), tau=1.0 / k)
    assert np.array_equal(Pi.cpu().numpy(), np.full((k, y.numel()), 1.0 / k, dtype=np.float32))


@pytest.mark.parametrize("kh,k,n", [(5, 5, 32767), (5, 5, 32769), (3, 2, 1_048_575), (3, 2, 1_050_000), (70, 3, 524_289)])
def test_validate_ranges(kh, k, n):
    """Node ranges of one chunk and of two, and of 2048 nodes with a short last one
    (bar as above, times 30 for sums of 1e6 terms: rounding errors add up like their root)."""
    g = np.random.default_rng(n)
    A, B = g.random((kh, n)).astype(np.float32), g.random((k, n)).astype(np.float32)
    v = otm.validate(to_dev(A), to_dev(B), threshold=0.05)
    a, b = A.astype(np.float64), B.astype(np.float64)
    ac, bc = a - a.mean(1, keepdims=True), b - b.mean(1, keepdims=True)
    rho = ac @ bc.T / np.sqrt((ac**2).sum(1))[:, None] / np.sqrt((bc**2).sum(1))[None]
    assert np.abs(v.rho.cpu().numpy() - rho).max() < 3e-11
    l1 = np.stack([np.abs(a[i] - b).mean(1) for i in range(kh)])
    assert rel(v.l1.cpu().numpy(), l1) < 3e-11
