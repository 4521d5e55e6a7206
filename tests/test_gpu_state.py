"""Snapshot and restore copy the ring levels that later steps read; the
weakly-synchronous 1D run marks ring slots by one bit pattern.  The operations
are the same either way, so every comparison is of bits."""
import math

import numpy as np
import pytest
import torch

from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def field(n):
    u0 = I.u0_powerlaw(n, max(2, n // 16), 5)
    u0 = u0 / np.max(np.abs(u0))
    return u0, I.dt_rule(2 * math.pi / n, 1.0, 0.02)


# (a ring of L + m - 1 + 64 slots: the live levels wrap around its end, start at
# its first slot, or are fewer than it keeps)
@pytest.mark.parametrize("at_step", [1, 2, 66, 67, 68, 69, 130, 137])
@pytest.mark.parametrize("order,L", [(2, 3), (4, 4)])
def test_restore_at_any_slot(gpu, order, L, at_step):
    print("restore", order, L, at_step, flush=True)
    N, P, nst = 4096, 32, 170
    u0, dt = field(N)
    kw = dict(n=N, p=P, order=order, L=L, nu=0.02, dt=dt, nsteps_max=nst, seed=7, dist=1)
    a = gpu.Stepper(**kw)
    a.set_fuse(24)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    a.run(u, s, at_step)
    snap = a.snapshot(u)
    a.run(u, s, nst - at_step)
    b = gpu.Stepper(**kw)                       # the same configuration, another context
    for st, fuse in ((a, 24), (a, 1), (b, 16)):
        v = torch.empty_like(u)
        st.set_fuse(fuse)
        st.restore(snap.clone() if st is b else snap, v)
        st.run(v, s, nst - at_step)
        assert torch.equal(u, v)


def test_restore_in_record_mode(gpu):
    N, P, nst = 2048, 16, 90
    u0, dt = field(N)
    st = gpu.Stepper(n=N, p=P, order=2, L=3, nu=0.02, dt=dt, nsteps_max=nst, seed=7, dist=0,
                     record=True, ckpt_every=20)
    u, s = dev(u0), torch.empty(N, dtype=torch.float64, device="cuda")
    st.run(u, s, 50)
    snap = st.snapshot(u)
    st.run(u, s, nst - 50)
    g, gnu = st.adjoint(u)
    v = torch.empty_like(u)
    st.restore(snap, v)
    st.run(v, s, nst - 50)
    g2, gnu2 = st.adjoint(v)
    assert torch.equal(u, v) and torch.equal(g, g2) and torch.equal(gnu, gnu2)


@pytest.mark.parametrize("L", [0, 1, 6])
def test_restore_3d(gpu, L):
    print("restore 3D", L, flush=True)
    n, p, nst = (20, 18, 24), (2, 3, 2), 2 * L + 12
    st = gpu.Stepper(dim=3, n=n, p=p, order=2, L=L, nu=0.05, dt=1e-4, nsteps_max=nst, seed=3)
    g = torch.Generator().manual_seed(1)
    u0 = torch.rand((3, n[2], n[1], n[0]), generator=g, dtype=torch.float64).cuda()
    zero, u, s = st.snapshot(u0), torch.empty_like(u0), torch.empty_like(u0)
    for first in (1, L + 1, 2 * L + 5):
        st.restore(zero, u)
        st.run(u, s, first)
        snap, v = st.snapshot(u), torch.empty_like(u)
        st.run(u, s, nst - first)
        st.restore(snap, v)
        st.run(v, s, nst - first)
        assert torch.equal(u, v)


@pytest.mark.parametrize("order,at", [(2, 0), (2, 255), (4, 1), (4, 254)])
def test_ws_edge_with_the_unset_bits(gpu, order, at):
    """An edge value with the bits of an empty slot is sent as another NaN, so
    the run ends and the NaN spreads by at most h points per step."""
    print("ws unset bits", order, at, flush=True)
    N, P, nst, h = 4096, 16, 20, order // 2
    u0, dt = field(N)
    st = gpu.Stepper(n=N, p=P, order=order, L=2, nu=0.02, dt=dt, nsteps_max=nst)
    x = 5 * 256 + at
    u = dev(u0)
    u.view(torch.int64)[x] = 0x7FF4A55E7ED0DEAD
    st.run_ws(u, nst)
    bad = torch.isnan(u).nonzero().flatten().cpu().numpy()
    assert bad.size > 0 and x in bad
    assert bad.min() >= x - h * nst and bad.max() <= x + h * nst
