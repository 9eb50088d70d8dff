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


@pytest.mark.parametrize("n,d,m", [(500, 500, 20), (10_000, 10_000, 120), (50_000, 50_000, 200), (100_000, 10_000, 100),
                                   (40_000, 10_000, 31), (300_000, 2_000, 16)])
def test_second_moment_scratch(n, d, m):
    """One layout, not the larger of two: the product C S and, past 16 MB by panels, S
    again, both padded to whole panels of 16 columns with room for two more; the parts of a
    column sum (a 4096 x m at most); by rows, two sums of m + 2 for at most 8192 shares of
    the entries."""
    pitch = (m + 2 + 15) // 16 * 16
    got = otm.lib().otm_m2_apply_workspace(n, d, m)
    small = 4 * _up(8 * n) + 4 * _up(8 * d) + _up(8 * m)
    if m >= 32 and n * m >= 2_000_000:
        most = 8 * pitch * (n + d + max(4096, n // 64 + 1)) + small
    else:
        most = 8 * m * (n + 4096) + 16 * 8192 * (m + 2) + small
    assert 8 * m * n <= got <= most + 2048
