"""The 3D step at any block widths (variant 1: by bricks, 9: by points, 0: by size)
at the block shapes where their splits can go wrong: blocks two points wide,
widths that split unevenly, a last brick of one point, thin and long blocks,
one block on an axis, and scalars up to the largest tile.  Fixed evaluation
order, so the bits are the oracle's (no tolerance)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [((4, 4, 4), (2, 2, 2)), ((6, 4, 2), (1, 2, 1)), ((30, 10, 8), (3, 1, 2)),
          ((13, 13, 13), (1, 1, 1)), ((26, 39, 13), (2, 3, 1)), ((36, 24, 24), (3, 2, 2)),
          ((2, 70, 9), (1, 2, 3)), ((130, 3, 5), (1, 1, 1)), ((66, 34, 18), (2, 2, 2)),
          ((10, 10, 300), (2, 2, 2)), ((100, 50, 25), (2, 1, 1))]


@pytest.mark.parametrize("n,p", SHAPES)
@pytest.mark.parametrize("nscal,stale", [(0, 0), (2, 0), (4, 1)])
def test_any_block_widths(gpu, n, p, nscal, stale):
    print("bricks", n, p, nscal, stale, flush=True)
    L, nst, nu = 3, 12, 0.01
    alpha = tuple(0.01 / (j + 1) for j in range(nscal))
    g = np.random.default_rng(sum(n) + nscal)
    u0 = g.uniform(-1, 1, (3 + nscal, n[2], n[1], n[0]))
    dt = 0.05 * min((2 * np.pi / max(n)) ** 2 / 0.02, 2 * np.pi / max(n))
    nf = 6 * p[0] * p[1] * p[2]
    k = oracle.delays(nst, nf, L, 2, 0, 11)
    ref = oracle.run3d(u0, n, p, L, nu, dt, k, nst, stale=bool(stale), alpha=alpha)
    st = gpu.Stepper(dim=3, n=n, p=p, order=2, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=11,
                     halo_mode=stale, alpha=alpha)
    u = torch.from_numpy(u0).cuda()
    s, snap = torch.empty_like(u), st.snapshot(u)
    for v in (0, 1, 9):
        st.set_variant(v)
        st.restore(snap, u)
        st.run(u, s, nst - 5)
        st.run(u, s, 5)
        assert np.array_equal(u.cpu().numpy(), ref), v
