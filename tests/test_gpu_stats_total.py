"""GPU test of the statistics pass's total at the edges of its two levels: one
workgroup (2048 elements), a group of 64, the first workgroup of a second group,
a full grid and a grid whose last group is short; called twice on one stream, so
the slots that the first call emptied serve the second.  The oracle sums
exactly; the kernel's fp64 sums of a few thousand exact squares per workgroup are
off by at most 2^-53 each per addition, and their total is rounded once, so 1e-14
bounds the relative difference.  An infinity in the last element, and in the
first, makes the sum non-finite."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import oracle  # noqa: E402
from paper_1910_02054_amd import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
W = 64 * 4 * 8          # gradient elements a workgroup reads per round


@pytest.mark.parametrize("n", [1, W, W + 1, 63 * W, 64 * W, 64 * W + 8, 65 * W - 5, 128 * W, 2048 * W, 2048 * W + 8,
                               3_000_017])
def test_statistics_total_at_the_edges_of_its_levels(n):
    import torch
    from paper_1910_02054_amd import binding as zb
    g16 = workloads.random_case(91, n)[0]
    dev = torch.from_numpy(g16.view(np.int16)).cuda().view(torch.float16)
    total, _ = oracle.local_stats(g16)
    exact = float(total) * 2.0 ** -48
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(2):
        s = zb.zero_shard_stats(dev)
        zb.zero_shard_stats_async(dev, out)
        assert abs(s / exact - 1.0) <= 1e-14 and out.item() == s, (n, s, exact)
    for where in (0, n - 1):
        dev[where] = float("inf")
        assert not np.isfinite(zb.zero_shard_stats(dev))
        dev[where] = 0.0
    assert np.isfinite(zb.zero_shard_stats(dev))
    print("[gpu-stats-total] n=%d rel %.1e" % (n, s / exact - 1.0), flush=True)
