"""Fused reverse sweep (one-wave regions, levels recomputed from every fourth
one): the same lambda bits as one reverse step per launch, over region sizes,
tile widths that are and are not multiples of the points per thread, segment
lengths around the groups of four levels, orders, halo modes and rounding modes.

grad nu is a compensated sum of the same terms in another order: a few roundings
of the sum, since lambda is u itself and the terms u * u_xx add up without much
cancellation; 1e-13 leaves a factor of 100."""
import math

import numpy as np
import pytest
import torch

from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu
MODES = {"plain": {}, "stale": {"halo_mode": 1}, "linear": {"adv_mode": 1, "adv_speed": 0.5}}


@pytest.mark.parametrize("P,W,order,L,steps,C,mode,arith", [
    (1, 64, 2, 3, 9, 4, "plain", 0),          # a region wraps a grid shorter than itself
    (64, 4, 2, 3, 26, 13, "plain", 0),        # one lane is a whole tile
    (64, 4, 4, 4, 26, 13, "plain", 1),
    (100, 7, 2, 2, 21, 6, "stale", 0),        # lanes of 4 and 3 points
    (37, 13, 4, 4, 33, 32, "plain", 0),
    (300, 1001, 2, 3, 66, 65, "plain", 0),    # 6 and 5 points
    (300, 1001, 4, 2, 35, 35, "linear", 1),
    (410, 1024, 2, 3, 103, 70, "plain", 0),   # 8 points
    (403, 1023, 4, 4, 41, 20, "stale", 0),    # 8 and 7 points
    (520, 1003, 2, 1, 50, 50, "linear", 0),   # 10 and 9 points
    (1024, 1024, 2, 3, 70, 66, "plain", 1),   # 10 and 9 points of aligned tiles
    (1024, 1024, 4, 4, 37, 36, "plain", 0),
])
def test_fused_reverse_bits(gpu, P, W, order, L, steps, C, mode, arith):
    N = P * W
    nu = 2e-3
    u0 = I.u0_powerlaw(N, max(2, N // 16), 3)
    u0 = u0 / np.max(np.abs(u0))
    dt = I.dt_rule(2 * math.pi / N, 1.0, nu)
    print("adjoint waves P %d W %d order %d L %d steps %d C %d %s arith %d"
          % (P, W, order, L, steps, C, mode, arith), flush=True)
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=dt, nsteps_max=steps, seed=7,
                     dist=order // 4, record=True, ckpt_every=C, arith=arith, **MODES[mode])
    u = torch.from_numpy(np.ascontiguousarray(u0)).cuda()
    s = torch.empty(N, dtype=torch.float64, device="cuda")
    st.run(u, s, steps)
    g, gnu = st.adjoint(u)
    st.set_adjoint_fuse(1)
    g1, gnu1 = st.adjoint(u)
    assert bool(torch.isfinite(g1).all())
    assert torch.equal(g, g1)
    assert abs(gnu.item() - gnu1.item()) <= 1e-13 * abs(gnu1.item())
