"""The FP64 dense products behind the orthonormal basis, at the edges of their
tiles: m around 16, 64, 112 and 128 columns, d from m itself over one and several
workgroups of rows to the shapes of the wide kernel (2 x 7 tiles per wave).

Bars: Q^T Q = I within 1e-13 per entry (Cholesky QR applied twice) and
Q Q^T Y = Y within 1e-12 relative, for well-conditioned Y."""
import numpy as np
import pytest
import torch

from gpu_util import dev, rel

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,m", [(1, 1), (15, 15), (16, 16), (17, 17), (64, 63), (65, 64), (200, 65), (255, 112),
                                 (257, 113), (259, 128), (1000, 16), (1023, 20), (1500, 129), (2051, 200), (40000, 16),
                                 (33001, 100), (20011, 200), (2048, 33),
                                 (2049, 33), (1024, 65), (1025, 65)])
def test_orthonormalize(d, m):
    g = torch.Generator().manual_seed(d + m)
    Y = torch.randn((d, m), dtype=torch.float64, generator=g)
    if d < 2 * m:
        Y += 3 * np.sqrt(m) * torch.eye(d, m, dtype=torch.float64)     # a square Gaussian is ill-conditioned
    Q = otm.orthonormalize(Y.to(dev())).cpu()
    assert (Q.T @ Q - torch.eye(m, dtype=torch.float64)).abs().max().item() < 1e-13
    assert rel((Q @ (Q.T @ Y)).numpy(), Y.numpy()) < 1e-12
