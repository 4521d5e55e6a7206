"""A 1D context's launches follow from its variant and steps per launch alone: what
the autotuner chose is chosen again on another context by at_set_variant and
at_set_fuse.  And every region kind that the estimate of a launch's time can
pick gives the bits of single steps (fixed order: no tolerance)."""
import math

import numpy as np
import pytest
import torch

from paper_1911_05769_amd import inputs as I

pytestmark = pytest.mark.gpu


def stepper(gpu, P, W, order, L=3, arith=0, nsteps=200, **kw):
    N, nu = P * W, 2e-3
    u0 = I.u0_powerlaw(N, max(2, min(N // 16, 4096)), 5)
    u0 = u0 / np.max(np.abs(u0))
    st = gpu.Stepper(n=N, p=P, order=order, L=L, nu=nu, dt=I.dt_rule(2 * math.pi / N, 1.0, nu),
                     nsteps_max=nsteps, seed=7, dist=order // 4, arith=arith, **kw)
    return st, torch.from_numpy(np.ascontiguousarray(u0)).cuda()


@pytest.mark.parametrize("P,W,order,arith", [
    (8, 128, 2, 0), (1024, 1024, 2, 0), (999, 1001, 4, 0), (4096, 1024, 4, 1), (3000, 96, 4, 0),
    (700, 17, 2, 0), (40, 9, 2, 0), (16384, 1024, 4, 0), (16384, 1024, 2, 0), (16384, 1024, 4, 1)])
def test_tuned_launches_have_a_name(gpu, P, W, order, arith):
    print("plan", P, W, order, arith, flush=True)
    tuned, u0 = stepper(gpu, P, W, order, arith=arith)
    s = tuned.autotune(u0, 60)
    assert tuned.query()[1] == s
    named, _ = stepper(gpu, P, W, order, arith=arith)
    named.set_variant(tuned.variant)
    if tuned.variant != 4:
        named.set_fuse(s)
    assert named.query()[1] == s and named.variant == tuned.variant
    for n in (1, 2, 7, s, s + 1, 2 * s - 1, 100, 131, 1000):
        assert tuned.launch_shape(n) == named.launch_shape(n), n
    print("  variant %d, %d steps:" % (tuned.variant, s), tuned.launch_shape(200), flush=True)


def test_launch_shape_refusals(gpu):
    st, _ = stepper(gpu, 8, 128, 2)
    with pytest.raises(gpu.AtError) as e:
        st.launch_shape(0)
    assert e.value.status == gpu.AT_ERR_ARG
    box = gpu.Stepper(dim=3, n=(16, 16, 16), p=(2, 2, 2), order=2, L=1, nu=0.01, dt=1e-4, nsteps_max=4)
    with pytest.raises(gpu.AtError) as e:
        box.launch_shape(1)
    assert e.value.status == gpu.AT_ERR_ARG
    whole, _ = stepper(gpu, 8, 128, 2)
    whole.set_variant(4)
    assert whole.launch_shape(150) == (150, 4, 4)
    st.set_fuse(1)
    assert st.launch_shape(150) == (1, 8, 4)
    rec, _ = stepper(gpu, 8, 128, 2, record=True, ckpt_every=30)
    rec.set_fuse(64)
    assert rec.launch_shape(150)[0] == 30


def test_every_kind_of_the_estimate(gpu):
    seen = set()
    for P, W, order, s, arith in [
            (20, 1000, 2, 64, 0), (256, 1024, 2, 50, 0), (260, 1002, 4, 16, 0), (300, 1000, 2, 64, 0),
            (1024, 1024, 2, 48, 0), (520, 2000, 2, 48, 1), (512, 1024, 4, 48, 0), (1024, 1024, 4, 48, 0),
            (999, 1001, 4, 60, 1), (1500, 1024, 4, 32, 0), (300, 4097, 4, 64, 0), (4096, 1000, 4, 40, 1),
            (16384, 1024, 4, 48, 0), (1025, 4096, 4, 64, 0), (3000, 1024, 2, 8, 0), (3000, 33, 4, 6, 0)]:
        st, u0 = stepper(gpu, P, W, order, arith=arith)
        st.set_fuse(s)
        got = []
        for fuse in (s, 1):
            st.set_fuse(fuse)
            if fuse > 1:
                shape = st.launch_shape(s)
                seen.add(shape[1:])
                print("kind", (P, W, order, s, arith), shape, flush=True)
                snap = st.snapshot(u0)
            u, t = torch.empty_like(u0), torch.empty_like(u0)
            st.restore(snap, u)
            st.run(u, t, s)
            st.run(u, t, 3)
            got.append(u)
        assert torch.equal(got[0], got[1]), (P, W, order, s, arith)
        st.close()
    assert seen >= {(p, 1) for p in (4, 6, 8, 10, 12, 16, 20, 24, 32)} | {(16, 4)}


def test_variants_take_the_steps_of_variant_0(gpu):
    """Tiles of 96 points at order 4: fewer steps of 16 points per thread pass the
    limit of a region of 256 threads, but the tuner chooses 48 of them."""
    st, _ = stepper(gpu, 3000, 96, 4, L=2)
    st.set_fuse(48)
    st.set_variant(1)
    assert st.query()[1] == 48 and st.launch_shape(48) == (48, 16, 1)


def batch(gpu, sizes, tile, order, arith=0, nsteps=140):
    nu = 2e-3
    ins, u0 = [], []
    for j, n in enumerate(sizes):
        u = I.u0_powerlaw(n, max(2, min(n // 16, 4096)), j)
        u = u / np.max(np.abs(u))
        ins.append(dict(n=n, p=n // tile, order=order, L=1 + j % 3, nu=nu,
                        dt=I.dt_rule(2 * math.pi / n, 1.0, nu), nsteps_max=nsteps, seed=j, dist=1, arith=arith))
        u0.append(torch.from_numpy(np.ascontiguousarray(u)).cuda())
    return gpu.Batch(ins), ins, u0


@pytest.mark.parametrize("sizes,tile,order", [([4096, 8192, 16384], 128, 2), ([1 << 18] * 36, 256, 4),
                                              ([1 << 16] * 20, 64, 4), ([1 << 18] * 60 + [4096] * 5, 256, 2)])
def test_tuned_batch_has_a_name(gpu, sizes, tile, order):
    print("batch plan", len(sizes), tile, order, flush=True)
    tuned, _, u0 = batch(gpu, sizes, tile, order)
    s = tuned.autotune(u0, 64)
    named, _, _ = batch(gpu, sizes, tile, order)
    named.set_variant(tuned.variant)
    named.set_fuse(s)
    for n in (1, 2, 7, s, s + 1, 2 * s, 100, 140):
        assert tuned.launch_shape(n) == named.launch_shape(n), n
    print("  variant %d, %d steps:" % (tuned.variant, s), tuned.launch_shape(140), flush=True)


def test_batch_at_32_points(gpu):
    """Variant 1 on a batch large enough for 32 points per thread at 64 steps, and 16
    at 8: every instance's standalone bits, also where a run is shorter than a launch."""
    b, ins, u0 = batch(gpu, [1 << 18] * 36 + [4096, 12288], 256, 4)
    refs = {}
    for j in (0, 17, 36, 37):
        st = gpu.Stepper(**dict(ins[j], fuse_steps=1))
        u = u0[j].clone()
        st.run(u, torch.empty_like(u), 135)
        refs[j] = u
    for fuse, points in ((64, 32), (8, 16)):
        b.reset()
        b.set_fuse(fuse)
        us = [u.clone() for u in u0]
        t = [torch.empty_like(u) for u in u0]
        assert b.launch_shape(128) == (min(64, fuse), points)
        b.run(us, t, 128, use_graph=True)
        b.run(us, t, 7)
        for j, ref in refs.items():
            assert torch.equal(us[j], ref), (fuse, j)
    with pytest.raises(gpu.AtError) as e:
        b.launch_shape(0)
    assert e.value.status == gpu.AT_ERR_ARG
