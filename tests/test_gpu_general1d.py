"""The general one-step kernel (k_step1d) at the tile widths that no other kernel
takes (2, 3, 5, 6 and 9 points; 4 points with long delays) and the delay bounds
up to the largest: at_init accepts them, so at_step and at_run have to step
them, by single steps and by the most steps per launch of the grid.  The
operations and their order are the oracle's, so the bits are."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu


def most_fused(st):
    for s in range(64, 0, -1):
        try:
            st.set_fuse(s)
            return s
        except Exception as e:
            assert "limit" in str(e)
    raise AssertionError("one step per launch refused")


@pytest.mark.parametrize("W,order", [(2, 2), (3, 2), (5, 2), (6, 2), (9, 2), (4, 4), (5, 4), (6, 4), (9, 4)])
@pytest.mark.parametrize("L", [0, 4, 15])
def test_widths_without_regions(gpu, W, order, L):
    for P in (1, 7, 2000):
        print("general", W, order, L, P, flush=True)
        N, nu, nst = P * W, 0.02, 40
        if N < 2 * order:
            continue                                  # a grid without modes
        u0 = I.u0_powerlaw(N, max(2, N // 16), 5)
        u0 = u0 / np.max(np.abs(u0))
        dt = I.dt_rule(2 * math.pi / N, 1.0, nu)
        k = oracle.delays(nst, 2 * P, L, order // 2 + 1, 0, 9)
        ref = oracle.run1d(u0, N, P, order, L, nu, dt, k, nst)
        st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=9, dist=0)
        u = torch.from_numpy(u0).cuda()
        s, snap = torch.empty_like(u), st.snapshot(u)
        for fuse in sorted({1, most_fused(st)}):
            st.set_fuse(fuse)
            st.restore(snap, u)
            st.run(u, s, nst - 3)
            a, b = u, s
            for _ in range(3):
                st.step(a, b)
                a, b = b, a
            assert np.array_equal(a.cpu().numpy(), ref, equal_nan=True), fuse
