"""The 3D point kernel (variant 9) on a box of so many planes that one launch of
a workgroup per plane would hold 2^32 threads: its launches together step the
whole box.  Fixed evaluation order, so the bits are the brick kernel's (variant
1; no tolerance)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_points_on_2_24_planes(gpu):
    n, p, steps = (2, 2, 1 << 24), (1, 1, 2), 3
    g = torch.Generator(device="cuda").manual_seed(5)
    u0 = torch.rand((3, n[2], n[1], n[0]), generator=g, dtype=torch.float64, device="cuda") - 0.5
    got = []
    for v in (1, 9):
        print("planes", n[2], "variant", v, flush=True)
        st = gpu.Stepper(dim=3, n=n, p=p, order=2, L=1, nu=0.01, dt=1e-9, nsteps_max=steps, seed=3)
        st.set_variant(v)
        u = u0.clone()
        s = torch.empty_like(u)
        st.run(u, s, steps - 1)
        st.step(u, s)
        got.append(s)
        st.close()
    assert bool(torch.isfinite(got[0]).all()) and not torch.equal(got[0], u0)
    assert torch.equal(got[0], got[1])
