"""The diagnostics reduction at the edges of its workgroup split: below one
workgroup, around one and several, where the workgroup count saturates, and
past it, against exactly rounded sums.

Tolerance: each partial is compensated (Neumaier), so the sums carry a few
roundings of the result whatever the order: 4 eps of sum |u| is allowed for
both sums (the mean divides it by n)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("n", [1, 63, 255, 257, 1023, 1025, 262145, 1024 * 1024 - 1,
                               1024 * 1024 + 257])
def test_stats_at_split_edges(gpu, n):
    print("stats", n, flush=True)
    g = np.random.default_rng(n)
    u = g.standard_normal(n) * np.exp(g.uniform(-20, 20, n))
    u[g.integers(n)] = -np.max(np.abs(u)) * 3.0
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    got = gpu.stats_noalloc(torch.from_numpy(u).cuda(), out).cpu().numpy()
    sabs = math.fsum(np.abs(u))
    assert got[0] == np.max(np.abs(u)) and got[3] == 0
    assert abs(got[2] - sabs) <= 4 * EPS * sabs
    assert abs(got[1] - math.fsum(u) / n) <= 4 * EPS * sabs / n
    # one non-finite value in the last place of the range
    v = u.copy()
    v[-1] = np.inf
    got = gpu.stats_noalloc(torch.from_numpy(v).cuda(), out).cpu().numpy()
    assert got[0] == np.inf and got[3] == 1
    v[-1] = np.nan
    got = gpu.stats_noalloc(torch.from_numpy(v).cuda(), out).cpu().numpy()
    assert math.isnan(got[0]) and got[3] == 1
