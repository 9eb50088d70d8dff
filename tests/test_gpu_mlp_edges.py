"""The warm-start perceptron's FP32 products at the batches where their kernel or its
tiles change: 1, 64 and 95 (64 x 64 tiles throughout the forward pass), 96 (the first
with 128 x 128 tiles), 128, 129 and 131 (a contraction over a batch that is no multiple
of 4), against float64 torch.

Bars: 2e-5 relative (2-norm) for outputs and gradients: float32 sums of 40400 terms
carry about sqrt(40400) 2^-24 = 1.2e-5 of their terms' norm."""
import pytest
import torch

from gpu_util import dev

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 64, 95, 96, 128, 129, 131])
def test_forward_backward(batch):
    dims = otm.ws_dims()
    ni, nh, no = dims["n_in"], dims["hidden"], dims["n_out"]
    g = torch.Generator(device=dev()).manual_seed(batch)
    r = lambda *s: torch.randn(s, device=dev(), generator=g)
    W1, b1, W2, b2 = r(nh, ni) / ni**0.5, 0.1 * r(nh), r(no, nh) / nh**0.5, 0.1 * r(no)
    params = torch.cat([x.reshape(-1) for x in (W1, b1, W2, b2)])
    X, dout = r(batch, ni), r(batch, no)
    H, out = otm.mlp_forward(params, X)
    grads = torch.zeros_like(params)
    otm.mlp_backward(params, X, H, dout, grads)
    torch.cuda.synchronize()
    d = lambda x: x.double()
    Z = d(X) @ d(W1).T + d(b1)
    near = (lambda a, b: ((d(a) - b).norm() / b.norm()).item())
    assert near(H, Z.clamp(min=0)) < 2e-5
    assert near(out, d(H) @ d(W2).T + d(b2)) < 2e-5
    dZ = (d(dout) @ d(W2)) * (H > 0)
    got = torch.split(grads, [nh * ni, nh, no * nh, no])
    for a, b in zip(got, (dZ.T @ d(X), dZ.sum(0), d(dout).T @ d(H), d(dout).sum(0))):
        assert near(a, b.reshape(-1)) < 2e-5
