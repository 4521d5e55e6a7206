"""The fused 1D kernels' regions at the tile widths and step counts where their
split of the grid can go wrong: widths that are one, two and a few threads of a
tile, widths no thread size divides (threads of p and p - 1 points), widths
without such a split, one tile, grids shorter than a region, and launches whose
rims take half a region.

The operations and their order are the oracle's, so the bits are (no
tolerance; a grid of 4 points diverges in both); the contracted mode has the
bits of its own one-step form."""
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


# tiles, width: 4 (one thread a tile), 5 (no split), 6 .. 9, around 16, 32 and
# 64 points, a few threads of p and p - 1 points, odd widths, one tile
SHAPES = [(40, 4), (30, 5), (20, 6), (33, 7), (64, 8), (7, 9), (30, 15), (25, 16), (40, 17),
          (6, 31), (9, 32), (5, 33), (11, 45), (3, 63), (8, 64), (4, 65), (300, 13), (37, 211),
          (3, 1001), (2, 2049), (1, 777), (1, 4), (1, 6), (2, 4096)]


@pytest.mark.parametrize("P,W", SHAPES)
@pytest.mark.parametrize("order,L,dist", [(2, 3, 0), (4, 4, 1)])
def test_widths(gpu, P, W, order, L, dist):
    print("widths", P, W, order, flush=True)
    N, nu, nst = P * W, 0.02, 71
    u0, dt = field(N, nu)
    k = oracle.delays(nst, 2 * P, L, order // 2 + 1, dist, 9)
    ref = oracle.run1d(u0, N, P, order, L, nu, dt, k, nst)
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=9, dist=dist)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    snap = st.snapshot(u)
    for v, fuse in [(0, 2), (0, 7), (0, 64), (1, 64), (2, 24), (3, 64)]:
        try:
            st.set_variant(v)
            st.set_fuse(fuse)
        except gpu.AtError:
            continue                     # this width takes no such variant or step count
        st.restore(snap, u)
        st.run(u, s, 40)                 # two runs: the second starts from the ring
        st.run(u, s, nst - 40)
        assert np.array_equal(u.cpu().numpy(), ref, equal_nan=True), (v, fuse)


@pytest.mark.parametrize("P,W", [(40, 17), (7, 129), (16, 64)])
@pytest.mark.parametrize("kw", [dict(halo_mode=1), dict(adv_mode=1, adv_speed=0.7), dict(L=15)])
def test_modes_on_odd_widths(gpu, P, W, kw):
    print("modes", P, W, kw, flush=True)
    N, nu, nst = P * W, 0.02, 50
    kw = dict(kw)
    L = kw.pop("L", 2)
    u0, dt = field(N, nu)
    k = oracle.delays(nst, 2 * P, L, 3, 1, 3)
    ref = oracle.run1d(u0, N, P, 4, L, nu, dt, k, nst, stale=kw.get("halo_mode") == 1,
                       linear=kw.get("adv_mode") == 1, adv_speed=kw.get("adv_speed", 0.0))
    st = gpu.Stepper(n=N, p=P, order=4, L=L, nu=nu, dt=dt, nsteps_max=nst, seed=3, dist=1,
                     fuse_steps=25, **kw)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    st.run(u, s, nst)
    assert np.array_equal(u.cpu().numpy(), ref)


@pytest.mark.parametrize("P,W", [(40, 17), (16, 64), (3, 1001)])
def test_contracted_and_recorded(gpu, P, W):
    """Contracted: fused launches have the bits of single steps.  Recorded: the
    adjoint's rebuild (every level stored) on odd widths, within 1e-12 of the
    oracle's gradient, the bound the adjoint is held to everywhere."""
    print("contracted, recorded", P, W, flush=True)
    N, nu, nst = P * W, 0.02, 45
    u0, dt = field(N, nu)
    got = []
    for fuse in (1, 45):
        st = gpu.Stepper(n=N, p=P, order=4, L=3, nu=nu, dt=dt, nsteps_max=nst, seed=3, dist=1,
                         arith=1, fuse_steps=fuse)
        u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
        st.run(u, s, nst)
        got.append(u)
    assert torch.equal(got[0], got[1])
    st = gpu.Stepper(n=N, p=P, order=2, L=3, nu=nu, dt=dt, nsteps_max=nst, seed=3, record=True,
                     ckpt_every=20, fuse_steps=64)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    st.run(u, s, nst)
    k = oracle.delays(nst, 2 * P, 3, 2, 0, 3)
    lam = np.cos(np.arange(N) * 0.37)
    g, gnu = st.adjoint(dev(lam))
    ref, gnu_ref = oracle.adjoint1d(u0, lam, N, P, 2, 3, nu, dt, k, nst)
    assert np.max(np.abs(g.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    assert abs(float(gnu) - gnu_ref) <= 1e-12 * max(abs(gnu_ref), float(np.sum(np.abs(lam))) * dt)


# grids large enough that the estimate of a launch's time picks 6, 10, 12, 20 and
# 24 points per thread, at tile widths that they divide and that they do not
@pytest.mark.parametrize("P,W,order,s,arith", [
    (256, 1024, 2, 50, 0), (260, 1002, 4, 16, 0), (1024, 1024, 2, 48, 0), (520, 2000, 2, 48, 1),
    (512, 1024, 4, 48, 0), (900, 768, 2, 30, 0), (1024, 1024, 4, 48, 0), (999, 1001, 4, 60, 1),
    (1024, 1000, 2, 64, 0), (4096, 1024, 4, 32, 0), (300, 4097, 4, 64, 0), (1000, 1200, 4, 48, 0)])
def test_points_per_thread(gpu, P, W, order, s, arith):
    print("points per thread", P, W, order, s, arith, flush=True)
    N, nu, nst = P * W, 2e-3, s + 3                  # two launches, of different length
    u0, dt = field(N, nu)
    st = gpu.Stepper(n=N, p=P, order=order, L=3, nu=nu, dt=dt, nsteps_max=nst, seed=2,
                     dist=order // 4, arith=arith)
    u, t = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    snap = st.snapshot(u)
    got = []
    for fuse in (1, s):
        st.set_fuse(fuse)
        st.restore(snap, u)
        st.run(u, t, nst)
        got.append(u.clone())
    assert torch.equal(got[0], got[1])


# runs on large grids take one launch more where their number would be odd, so
# that the last one writes the caller's field; a run of one step copies
@pytest.mark.parametrize("steps,fuse", [(1, 8), (2, 8), (7, 8), (20, 8), (24, 8), (50, 20), (61, 20), (3, 1)])
def test_even_number_of_launches(gpu, steps, fuse):
    print("even launches", steps, fuse, flush=True)
    N, P, nu = 1 << 21, 2048, 2e-3
    u0, dt = field(N, nu)
    st = gpu.Stepper(n=N, p=P, order=2, L=3, nu=nu, dt=dt, nsteps_max=2 * steps, seed=4)
    snap, got = st.snapshot(dev(u0)), []
    for f in (1, fuse):
        u, t = torch.empty(N, dtype=torch.float64, device="cuda"), torch.empty(N, dtype=torch.float64, device="cuda")
        st.set_fuse(f)
        st.restore(snap, u)
        if f == 1:
            for _ in range(2 * steps):
                st.step(u, t)
                u, t = t, u
        else:
            st.run(u, t, steps)
            st.run(u, t, steps)
        got.append(u)
    if fuse > 1:
        assert torch.equal(got[0], got[1])
    else:
        st.restore(snap, got[1])
        st.run(got[1], t, 2 * steps)
        assert torch.equal(got[0], got[1])
