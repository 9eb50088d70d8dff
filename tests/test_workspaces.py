"""Workspace sizes that callers plan with (host arithmetic only; no GPU)."""
import os

import pytest

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.skipif(not os.path.exists(otm.LIB_PATH), reason="library not built")


def _up(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("kh,k", [(1, 1), (10, 10), (64, 64), (65, 64), (100, 100), (128, 128), (16384, 1)])
def test_validation_scratch_is_bounded(kh, k):
    """The two arrays of partial sums hold a value per pair and node range: as many ranges as
    give two workgroups a CU (512 over the 64 x 64 tiles of pairs), and past that at most
    twice as many as 2048 nodes to each make.  The ranges are a grid's third dimension:
    at most 65535, at 134 million nodes."""
    m, tiles = kh * k, -(-kh // 64) * -(-k // 64)
    for n in (3, 64, 500, 5000, 50000, 10**6, 25_200_000, 65535 * 2048):
        got = otm.lib().otm_validate_workspace(kh, k, n) - 2 * _up(8 * (kh + k)) - _up(4 * m)
        most = min(65535, max(2 * -(-n // 2048), -(-512 // tiles)))
        assert 2 * _up(8 * m * -(-n // 2048)) <= got <= 2 * _up(8 * m * most), n
