"""Every narrow and odd tile width in launches that do take place: at each width
single steps and the most steps per launch of the grid (and some between, cut
to that limit) with every points-per-thread variant whose points divide the
width, against the oracle bit for bit; then the adjoint, whose forward rebuild
fuses up to 64 steps at any width, against the oracle's gradient."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def field(n, nu, seed=5):
    u0 = I.u0_powerlaw(n, max(2, n // 16), seed)
    u0 = u0 / np.max(np.abs(u0))
    return u0, I.dt_rule(2 * math.pi / n, 1.0, nu)


def limit(gpu, st):
    """The most steps per launch st takes."""
    for s in range(64, 1, -1):
        try:
            st.set_fuse(s)
            return s
        except gpu.AtError as e:
            assert e.status == gpu.AT_ERR_ARG
    return 1


# tiles, width: one thread a tile (4, 8, 16, 32), threads of p and p - 1 points
# (7, 10, 11, 13, 17, ...), no split (6, 9), a grid shorter than a region, one tile
SHAPES = [(40, 4), (1, 4), (20, 6), (33, 7), (64, 8), (7, 9), (9, 10), (13, 11), (50, 12), (300, 13),
          (30, 15), (25, 16), (40, 17), (90, 20), (11, 21), (6, 31), (9, 32), (5, 33), (11, 45), (3, 63), (8, 64), (4, 65),
          (37, 211), (1, 777), (3, 1001)]


@pytest.mark.parametrize("P,W", SHAPES)
@pytest.mark.parametrize("order,L,dist", [(2, 3, 0), (4, 4, 1), (4, 1, 0)])
def test_every_width_steps(gpu, P, W, order, L, dist):
    print("widths", P, W, order, L, flush=True)
    N, nu, nst = P * W, 0.02, 71
    u0, dt = field(N, nu)
    k = oracle.delays(nst, 2 * P, L, order // 2 + 1, dist, 9)
    ref = oracle.run1d(u0, N, P, order, L, nu, dt, k, nst)
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=9, dist=dist)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    snap = st.snapshot(u)
    ran = 0
    for v, points in ((0, 1), (1, 16), (2, 8), (3, 4)):
        if W % points != 0:
            with pytest.raises(gpu.AtError):
                st.set_variant(v)
            continue
        st.set_variant(v)
        most = limit(gpu, st)
        for fuse in sorted({min(f, most) for f in (1, 2, 7, 24, 64)}):
            st.set_fuse(fuse)
            st.restore(snap, u)
            st.run(u, s, 40)                     # two runs: the second starts from the ring
            st.run(u, s, nst - 40)
            assert np.array_equal(u.cpu().numpy(), ref, equal_nan=True), (v, fuse)
            ran += fuse
    assert ran > 1 or limit(gpu, st) == 1


@pytest.mark.parametrize("P,W", [(40, 4), (33, 7), (64, 8), (13, 11), (40, 17), (5, 33), (3, 63), (1, 777)])
@pytest.mark.parametrize("order,L", [(2, 3), (4, 4)])
def test_gradient_on_narrow_widths(gpu, P, W, order, L):
    """Segments of 66 steps: the rebuild runs launches of up to 64 steps.  The
    bound is the one the adjoint is held to everywhere."""
    print("gradient", P, W, order, flush=True)
    N, nu, nst = P * W, 0.02, 70
    u0, dt = field(N, nu)
    dt *= 0.2                                    # (the shortest grids stay finite)
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=3, dist=0,
                     record=True, ckpt_every=66)
    u = dev(u0)
    st.run(u, torch.empty_like(u), nst)
    k = oracle.delays(nst, 2 * P, L, order // 2 + 1, 0, 3)
    lam = np.cos(np.arange(N) * 0.37)
    ref, gnu_ref = oracle.adjoint1d(u0, lam, N, P, order, L, nu, dt, k, nst)
    assert np.all(np.isfinite(ref))
    g, gnu = st.adjoint(dev(lam))
    assert np.max(np.abs(g.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    assert abs(float(gnu) - gnu_ref) <= 1e-12 * max(abs(gnu_ref), float(np.sum(np.abs(lam))) * dt)
