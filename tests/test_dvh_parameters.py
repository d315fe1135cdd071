"""Doses to the hottest voxels from histograms: against the sorted bins, for empty,
one-bin, sparse and full rows and any rank (outside 1 .. N it is clamped)."""
import numpy as np
import pytest

from paper_2512_18863_amd.plan_eval import d_from_histogram, dvh_parameters


@pytest.mark.parametrize("n_bins,fill", [(0, 0), (1, 0), (1, 3), (7, 0), (7, 1), (40, 1), (40, 5), (3000, 2)])
def test_hottest(n_bins, fill):
    rng = np.random.default_rng(n_bins + fill)
    row = rng.integers(0, fill + 1, size=n_bins).astype(np.int64)
    voxels = np.repeat(np.arange(n_bins), row)[::-1]  # bins, hottest voxel first
    n = len(voxels)
    for k in (-2, 0, 1, 2, n // 2, n - 1, n, n + 4):
        want = voxels[min(max(k, 1), n) - 1] * 0.05 if n else 0.0
        assert d_from_histogram(row, 0.05, k) == want
    if n:
        got = dvh_parameters(row, (n, 1.0, 2.0), 0.05, 0.3, 1)
        for key, k in (("D98", (98 * n + 99) // 100), ("D50", (50 * n + 99) // 100), ("D2", (2 * n + 99) // 100),
                       ("D2cc", 7)):
            assert got[key] == voxels[min(max(k, 1), n) - 1] * 0.05
