"""The whole-grid variant in launches that go around the ring of L + m - 1 + 64
edge levels more than once: the levels it leaves there are the last ones, in
their slots, so that ordinary steps continue from them bit for bit."""
import math

import numpy as np
import pytest
import torch

from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,order,L", [(1024, 8, 2, 3), (1360, 5, 4, 4), (4096, 256, 2, 2)])
@pytest.mark.parametrize("steps", [63, 70, 139, 141, 300])
def test_long_launch_then_single_steps(gpu, N, P, order, L, steps):
    print("whole", N, P, order, L, steps, flush=True)
    u0 = I.u0_powerlaw(N, max(2, N // 16), 5)
    u0 = u0 / np.max(np.abs(u0))
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=0.02, dt=I.dt_rule(2 * math.pi / N, 1.0, 0.02),
                     nsteps_max=steps + 20, seed=7, dist=1)
    u = torch.from_numpy(np.ascontiguousarray(u0)).cuda()
    s, zero = torch.empty_like(u), st.snapshot(u)
    got = []
    for v in (4, 0):
        st.set_variant(v)
        if v == 0:
            st.set_fuse(1)
        st.restore(zero, u)
        st.run(u, s, steps)
        st.set_variant(0)
        st.set_fuse(1)
        st.run(u, s, 20)
        got.append(u.clone())
    assert torch.equal(got[0], got[1])
