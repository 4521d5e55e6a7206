"""The work a user of the AT Burgers stepper has it do, as a set of measured cases.

Each case is one pass through the public entry points of
``paper_1911_05769_amd`` (``at.Stepper``, ``at.Batch``, ``autograd``): a run
restarted from a snapshot, a user's own step-by-step loop with diagnostics, a
batch of instances, a gradient through the adjoint, a weakly-synchronous run.
``exact`` evaluates the same scheme in plain torch (binary64): central
differences and forward Euler, with the halo values across tile or block faces
extrapolated in time from the delayed levels.

The sizes are those of the benchmark's workloads (with fewer steps for the
largest), of the paper's own 3D runs, and generic odd ones.
"""
import math

import torch

from paper_1911_05769_amd import at
from paper_1911_05769_amd import autograd as AG

TWO_PI = 2.0 * math.pi
UNIFORM, HALF_ZERO = at.DIST_UNIFORM, at.DIST_HALF_ZERO


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _run1d(name, tiles, width, order, L, steps, nu, arith=0, mode="burgers"):
    return {"name": name, "kind": "run1d", "tiles": tiles, "width": width, "order": order, "L": L,
            "steps": steps, "nu": nu, "arith": arith, "mode": mode}


def _run3d(name, n, blocks, L, steps, scalars):
    return {"name": name, "kind": "run3d", "nx": n[0], "ny": n[1], "nz": n[2], "bx": blocks[0],
            "by": blocks[1], "bz": blocks[2], "L": L, "steps": steps, "scalars": scalars}


def listed():
    return [
        # the smallest grid of the benchmark: 8 KB of state, every step is latency
        _run1d("run1d_small", 8, 128, 2, 2, 1000, 0.05),
        # a run of a million points: it fits the caches, one launch is short
        _run1d("run1d_mid", 1024, 1024, 2, 3, 1000, 2e-3),
        # the same size on tiles of an odd width (a grid cut by its users' decomposition)
        _run1d("run1d_ragged", 999, 1001, 4, 4, 500, 2e-3),
        # the headline run: 2^24 points, 4th order, arithmetic in the fixed order
        _run1d("run1d_large", 4096, 4096, 4, 4, 500, 1e-3),
        # a production run that does not need bit-reproducibility against the fixed order
        _run1d("run1d_contracted", 4096, 1024, 4, 4, 500, 1e-3, arith=1),
        # a user's own time loop: single steps, a blow-up check after every few
        {"name": "step_and_check", "kind": "loop1d", "tiles": 300, "width": 1000, "order": 2,
         "L": 3, "rounds": 16, "per_round": 4, "nu": 5e-3},
        # a parameter study: many independent instances of uneven size together
        {"name": "batch_study", "kind": "batch", "count": 256, "log2_lo": 12.0, "log2_hi": 18.0,
         "tile": 256, "order": 4, "steps": 500, "arith": 0},
        # one gradient of a misfit with respect to u0 and nu (data assimilation)
        {"name": "gradient", "kind": "gradient", "tiles": 1024, "width": 1024, "order": 2, "L": 3,
         "steps": 1000, "ckpt": 100, "nu": 2e-3},
        # the weakly-synchronous run: tiles advance on their own, delays emerge
        {"name": "weakly_sync", "kind": "ws1d", "tiles": 1024, "width": 1024, "order": 2, "L": 3,
         "steps": 500, "nu": 2e-3},
        # the largest box: 512^3 in 8^3 blocks, 3.2 GB per level
        _run3d("box_large", (512, 512, 512), (8, 8, 8), 3, 20, 0),
        # the paper's own case: 120^3 on 1000 processes of 12^3, L = 10
        _run3d("box_paper", (120, 120, 120), (10, 10, 10), 10, 100, 0),
        # a box with two passive scalars
        _run3d("box_scalars", (256, 256, 256), (4, 4, 4), 3, 20, 2),
    ]


def _logu(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _tiles(rng, lo, hi):
    """(tiles, width) with lo <= tiles*width <= hi, any width from 16 to 8192."""
    n = _logu(rng, lo, hi)
    w = int(_logu(rng, 16, min(8192, n)))
    if rng.random() < 0.5:                  # half of the grids have round widths
        w = max(16, w // 16 * 16)
    return max(1, int(n / w)), w


def draw(rng):
    kind = rng.choice(["run1d", "run1d", "run1d", "loop1d", "batch", "gradient", "ws1d", "run3d",
                       "run3d"])
    order = rng.choice([2, 4])
    L = rng.choice([0, 1, 2, 3]) if order == 2 else rng.choice([1, 2, 4])
    nu = round(_logu(rng, 1e-3, 5e-2), 5)
    if kind == "run1d":
        t, w = _tiles(rng, 512, 1 << 24)
        steps = int(max(20, min(1000, 4e9 / (t * w))))
        c = _run1d("", t, w, order, L, rng.randint(steps // 2, steps), nu,
                   arith=rng.choice([0, 0, 1]), mode=rng.choice(["burgers"] * 4 + ["linear"]))
    elif kind == "loop1d":
        t, w = _tiles(rng, 512, 1 << 22)
        c = {"kind": kind, "tiles": t, "width": w, "order": order, "L": L,
             "rounds": rng.randint(4, 16), "per_round": rng.randint(1, 8), "nu": nu}
    elif kind == "batch":
        lo = rng.uniform(9.0, 13.0)
        c = {"kind": kind, "count": int(_logu(rng, 4, 256)), "log2_lo": round(lo, 2),
             "log2_hi": round(lo + rng.uniform(1.0, 5.0), 2), "tile": rng.choice([64, 128, 256]),
             "order": order, "steps": rng.randint(100, 400), "arith": rng.choice([0, 0, 1])}
    elif kind == "gradient":
        n = _logu(rng, 1024, 1 << 20)
        w = int(_logu(rng, 16, min(4096, n)))
        w = w if rng.random() < 0.25 else max(16, w // 16 * 16)
        c = {"kind": kind, "tiles": max(1, int(n / w)), "width": w, "order": order, "L": L,
             "steps": rng.randint(100, 500), "ckpt": rng.choice([20, 50, 100]), "nu": nu}
    elif kind == "ws1d":
        c = {"kind": kind, "tiles": int(_logu(rng, 64, 1024)),
             "width": rng.choice([256, 512, 1024, 2048]), "order": order, "L": L,
             "steps": rng.randint(100, 500), "nu": nu}
    else:
        s = rng.choice([0, 0, 0, 1, 2, 4])
        if rng.random() < 0.5:              # blocks of 64-point multiples in x
            b = [rng.randint(1, 4), rng.randint(1, 8), rng.randint(1, 6)]
            n = [64 * b[0] * rng.randint(1, 2), b[1] * 8 * rng.randint(1, 6),
                 b[2] * rng.randint(6, 48)]
        else:                               # any block widths
            b = [rng.randint(1, 10), rng.randint(1, 10), rng.randint(1, 10)]
            n = [q * rng.randint(5, 32) for q in b]
        c = _run3d("", n, b, rng.choice([0, 1, 3, 6]), rng.randint(10, 60), s)
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _dt(dx, nu):
    """The time step rule of the workloads, max|u0| = 1."""
    return 0.2 * min(dx, dx * dx / (2.0 * nu))


def _field1d(n, seed, modes=12):
    """Multi-scale sinusoidal field: random-phase modes kappa <= n/16 with
    amplitude kappa^-2 (kappa = 1 among them), scaled to max|u| = 1."""
    g = torch.Generator().manual_seed(seed)
    top = max(2.0, n / 16.0)
    kap = torch.exp(torch.rand(modes, generator=g, dtype=torch.float64) * math.log(top)).floor()
    kap[0] = 1.0
    th = torch.rand(modes, generator=g, dtype=torch.float64) * TWO_PI
    x = torch.arange(n, dtype=torch.float64, device="cuda") * (TWO_PI / n)
    u = torch.zeros_like(x)
    for k, t in zip(kap.tolist(), th.tolist()):
        u += k ** -2.0 * torch.cos(k * x + t)
    return u / u.abs().max()


def _field3d(c, seed, modes=6):
    """Divergence-free sum of random-phase modes plus the scalars, each
    scaled to max 1: [3 + scalars][nz][ny][nx]."""
    g = torch.Generator().manual_seed(seed)
    nc = 3 + c["scalars"]
    out = torch.zeros((nc, c["nz"], c["ny"], c["nx"]), dtype=torch.float64, device="cuda")
    ax = [torch.arange(c[k], dtype=torch.float64, device="cuda") * (TWO_PI / c[k])
          for k in ("nx", "ny", "nz")]
    for _ in range(modes):
        k = torch.randint(-4, 5, (3,), generator=g).double()
        k[0] = k[0] if k.abs().sum() > 0 else 1.0
        a = torch.randn(nc, generator=g, dtype=torch.float64)
        a[:3] -= k * ((a[:3] @ k) / (k @ k))
        a *= float(k @ k) ** (-11.0 / 12.0)
        th = float(torch.rand(1, generator=g)) * TWO_PI
        phase = (k[2].item() * ax[2])[:, None, None] + (k[1].item() * ax[1])[None, :, None] + \
            (k[0].item() * ax[0])[None, None, :] + th
        m = torch.cos(phase)
        for j in range(nc):
            out[j] += a[j].item() * m
    out[:3] /= out[:3].abs().max()
    for j in range(3, nc):
        out[j] /= out[j].abs().max()
    return out


def _dist(order):
    return UNIFORM if order == 2 else HALF_ZERO


NU3 = 5e-3


def _alpha(c):
    return tuple(NU3 / (1.0 + j) for j in range(c["scalars"]))


def _dt3(c):
    return min(_dt(TWO_PI / c[k], NU3) for k in ("nx", "ny", "nz"))


def _instances(c, seed):
    """The batch's instances, as plain values: the sizes and viscosities of the
    study are the case's, the initial fields and delays the seed's."""
    g = torch.Generator().manual_seed(c["count"])
    r = torch.rand((c["count"], 3), generator=g, dtype=torch.float64).tolist()
    got = []
    for j, (a, b, d) in enumerate(r):
        size = 2.0 ** (c["log2_lo"] + a * (c["log2_hi"] - c["log2_lo"]))
        n = c["tile"] * max(1, round(size / c["tile"]))
        nu = 1e-3 * 100.0 ** b
        got.append(dict(n=n, p=n // c["tile"], order=c["order"], L=(1, 2, 4)[int(3 * d)] if
                        c["order"] == 4 else (1, 2, 3)[int(3 * d)], nu=nu, dt=_dt(TWO_PI / n, nu),
                        nsteps_max=c["steps"], seed=seed + j, dist=HALF_ZERO, arith=c["arith"]))
    return got


def _stepper1d(c, seed, steps, **kw):
    n = c["tiles"] * c["width"]
    linear = c.get("mode") == "linear"
    return at.Stepper(n=n, p=c["tiles"], order=c["order"], L=c["L"], nu=c["nu"],
                      dt=_dt(TWO_PI / n, c["nu"]), nsteps_max=steps, seed=seed,
                      dist=_dist(c["order"]), adv_mode=1 if linear else 0,
                      adv_speed=0.8 if linear else 0.0, **kw)


def prepare(case, seed):
    c, s = case, {"case": case}
    if c["kind"] in ("run1d", "loop1d", "ws1d"):
        steps = c["rounds"] * c["per_round"] if c["kind"] == "loop1d" else c["steps"]
        st = _stepper1d(c, seed, steps, arith=c.get("arith", 0))
        u = _field1d(c["tiles"] * c["width"], seed)
        if c["kind"] == "run1d":
            st.autotune(u, min(steps, 100))
        s.update(st=st, u=u, scratch=torch.empty_like(u), snap=st.snapshot(u))
    elif c["kind"] == "batch":
        ins = _instances(c, seed)
        b = at.Batch(ins)
        sizes = [i["n"] for i in ins]
        u0 = torch.cat([_field1d(i["n"], i["seed"], modes=6) for i in ins])
        u, scr = torch.empty_like(u0), torch.empty_like(u0)
        us = list(torch.split(u, sizes))
        b.autotune(list(torch.split(u0, sizes)), min(c["steps"], 128))
        s.update(b=b, u0=u0, u=u, us=us, scratch=list(torch.split(scr, sizes)))
    elif c["kind"] == "gradient":
        n = c["tiles"] * c["width"]
        spec = AG.StepSpec(n=n, p=c["tiles"], order=c["order"], L=c["L"],
                           dt=_dt(TWO_PI / n, c["nu"]), nsteps=c["steps"], ckpt_every=c["ckpt"],
                           seed=seed, dist=_dist(c["order"]))
        s.update(spec=spec, u0=_field1d(n, seed).requires_grad_(True),
                 nu=torch.tensor(c["nu"], dtype=torch.float64, requires_grad=True),
                 target=_field1d(n, seed + 1000003))
    else:
        st = at.Stepper(dim=3, n=(c["nx"], c["ny"], c["nz"]), p=(c["bx"], c["by"], c["bz"]),
                        order=2, L=c["L"], nu=NU3, dt=_dt3(c), nsteps_max=c["steps"], seed=seed,
                        dist=UNIFORM, alpha=_alpha(c))
        u = _field3d(c, seed)
        st.autotune(u, 4)
        s.update(st=st, u=u, scratch=torch.empty_like(u), snap=st.snapshot(u))
    return s


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind in ("run1d", "run3d"):
        st, u = state["st"], state["u"]
        st.restore(state["snap"], u)
        st.run(u, state["scratch"], c["steps"])
        return u
    if kind == "loop1d":
        st, a, b = state["st"], state["u"], state["scratch"]
        st.restore(state["snap"], a)
        checks = []
        for _ in range(c["rounds"]):
            for _ in range(c["per_round"]):
                st.step(a, b)
                a, b = b, a
            checks.append(st.stats(a))
        return {"u": a, "checks": checks}
    if kind == "ws1d":
        st, u = state["st"], state["u"]
        st.restore(state["snap"], u)
        st.run_ws(u, c["steps"])
        return u
    if kind == "batch":
        state["u"].copy_(state["u0"])
        state["b"].reset()
        state["b"].run(state["us"], state["scratch"], c["steps"], use_graph=True)
        return state["u"]
    u0, nu = state["u0"], state["nu"]
    u0.grad = nu.grad = None
    uT = AG.AtBurgers.apply(u0, nu, state["spec"])
    J = AG.AtMisfit.apply(uT, state["target"])
    J.backward()
    return {"u": uT.detach(), "J": J.detach(), "du0": u0.grad, "dnu": nu.grad}


def work(case):
    """Bytes: the fields in and out and the delays, once; flops: the scheme's."""
    c, kind = case, case["kind"]
    if kind == "run3d":
        npt, nc = c["nx"] * c["ny"] * c["nz"], 3 + c["scalars"]
        faces = 6 * c["bx"] * c["by"] * c["bz"]
        return {"bytes": 16.0 * nc * npt + faces * c["steps"],
                "flops": 29.0 * nc * npt * c["steps"]}
    if kind == "batch":
        ins = _instances(c, 1)
        pts, faces = sum(i["n"] for i in ins), sum(2 * i["p"] for i in ins)
        per = 17.0 if c["order"] == 4 else 11.0
        return {"bytes": 16.0 * pts + faces * c["steps"], "flops": per * pts * c["steps"]}
    n = float(c["tiles"] * c["width"])
    steps = c["rounds"] * c["per_round"] if kind == "loop1d" else c["steps"]
    per = 17.0 if c["order"] == 4 else 11.0
    if kind == "loop1d":        # every level is the user's: read, written, and read by the checks
        return {"bytes": 16.0 * n * steps + 8.0 * n * c["rounds"],
                "flops": per * n * steps + 4.0 * n * c["rounds"]}
    if kind == "gradient":      # forward, its recomputation and the transpose
        return {"bytes": 32.0 * n + 2.0 * c["tiles"] * steps, "flops": (2 * per + 30.0) * n * steps}
    return {"bytes": 16.0 * n + 2.0 * c["tiles"] * steps, "flops": per * n * steps}


# ---------------------------------------------------------------------------
# the scheme in plain torch
# ---------------------------------------------------------------------------

def _delays(steps, faces, L, m, dist, seed):
    """k[n][f]: SplitMix64 of seed + gamma*(1 + n*F + f) mapped to the
    distribution, then min(k, max(0, n - m + 1))."""
    M = (1 << 64) - 1

    def s64(v):                         # the int64 with the same bits
        v &= M
        return v - (1 << 64) if v >> 63 else v

    def shr(z, b):                      # logical shift
        return (z >> b) & ((1 << (64 - b)) - 1)

    i = torch.arange(1, steps * faces + 1, dtype=torch.int64, device="cuda")
    z = i * s64(0x9E3779B97F4A7C15) + s64(seed)
    z = (z ^ shr(z, 30)) * s64(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * s64(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    hi, lo = shr(z, 32), z & 0xFFFFFFFF
    if dist == UNIFORM:
        k = (hi * (L + 1)) >> 32
    else:
        k = torch.where(lo < (1 << 31), torch.zeros_like(hi), 1 + ((hi * L) >> 32))
        k = k if L > 0 else torch.zeros_like(k)
    k = k.reshape(steps, faces)
    lim = (torch.arange(steps, device="cuda") - (m - 1)).clamp(min=0)
    return torch.minimum(k, lim[:, None])


class _Tiled:
    """Concatenated periodic 1D instances cut into tiles: index tables, and
    one step of the scheme on the whole vector."""

    def __init__(self, ins):
        self.order = ins[0]["order"]
        self.h, self.m = self.order // 2, 2 if self.order == 2 else 3
        h = self.h
        pos, start, left, right, cols, at0, t0 = [], [], [], [], [], 0, 0
        per = {k: [] for k in ("nu", "dt", "c1", "c2")}
        delays = []
        for q in ins:
            n, p = q["n"], q["p"]
            i = torch.arange(n, device="cuda")
            pos.append(torch.stack([(i + d) % n + at0 for d in range(-h, h + 1)]))
            t = torch.arange(p, device="cuda")
            start.append(at0 + t * (n // p))
            left.append(t0 + (t - 1) % p)
            right.append(t0 + (t + 1) % p)
            cols.append(torch.full((p,), n // p, device="cuda"))
            dx = TWO_PI / n
            w = 1.0 if self.order == 2 else 12.0
            for k, v in (("nu", q["nu"]), ("dt", q["dt"]),
                         ("c1", 1.0 / ((2.0 if w == 1.0 else w) * dx)), ("c2", 1.0 / (w * dx * dx))):
                per[k].append(v if len(ins) == 1 else
                              torch.full((n,), v, dtype=torch.float64, device="cuda"))
            delays.append(_delays(q["nsteps_max"], 2 * p, q["L"], self.m, q["dist"], q["seed"])
                          .reshape(-1, p, 2).to(torch.int8))
            at0, t0 = at0 + n, t0 + p
        self.pos = torch.cat(pos, 1)
        start, end = torch.cat(start), torch.cat(start) + torch.cat(cols)
        self.left, self.right = torch.cat(left), torch.cat(right)
        e = torch.arange(h, device="cuda")
        # the edge points [tile][side][q], left to right
        self.edge = torch.stack([start[:, None] + e, end[:, None] - h + e], 1)
        self.coef = {k: v[0] if len(ins) == 1 else torch.cat(v) for k, v in per.items()}
        self.delays = torch.cat(delays, 1)
        self.depth = max(q["L"] for q in ins) + self.m
        self.cadv = ins[0].get("cadv")

    def halos(self, hist, n):
        """hist: edges of levels n, n-1, ... [depth][T][2][h] -> [T][2][h]."""
        k = self.delays[n].long()
        T = k.shape[0]
        src = torch.stack([self.left, self.right], 1)              # the tile across each face
        side = torch.tensor([1, 0], device="cuda").expand(T, 2)
        v = [hist[(k + j).clamp(max=hist.shape[0] - 1), src, side] for j in range(self.m)]
        kk = k.double()[:, :, None]
        d1 = v[0] - v[1]
        if self.m == 2:
            hv = v[0] + kk * d1
        else:
            hv = (v[0] + kk * d1) + 0.5 * kk * (kk + 1.0) * (d1 - (v[1] - v[2]))
        return torch.where(k[:, :, None] == 0, v[0], hv)

    def step(self, u, hist, n, nu=None):
        """u, hist (edges of levels n-1, ...) -> level n+1, hist with level n."""
        h = self.h
        hist = torch.cat([u[self.edge][None], hist])[: self.depth]
        hv = self.halos(hist, n)
        nb = [u[self.pos[j]] for j in range(2 * h + 1)]
        for d in range(1, h + 1):                       # neighbours at distance d
            for j in range(d):                          # edge point j reads across the face
                nb[h - d] = nb[h - d].index_put((self.edge[:, 0, j],), hv[:, 0, h - d + j])
                nb[h + d] = nb[h + d].index_put((self.edge[:, 1, h - 1 - j],),
                                                hv[:, 1, d - 1 - j])
        c = self.coef
        if self.order == 2:
            D1 = (nb[2] - nb[0]) * c["c1"]
            D2 = ((nb[2] - 2.0 * u) + nb[0]) * c["c2"]
        else:
            D1 = (8.0 * (nb[3] - nb[1]) - (nb[4] - nb[0])) * c["c1"]
            D2 = ((16.0 * (nb[3] + nb[1]) - 30.0 * u) - (nb[4] + nb[0])) * c["c2"]
        a = u if self.cadv is None else self.cadv
        F = (c["nu"] if nu is None else nu) * D2 - a * D1
        return u + c["dt"] * F, hist

    def first(self, u):
        return torch.zeros((self.depth,) + tuple(self.edge.shape), dtype=torch.float64,
                           device="cuda")


def _tiled1d(c, seed, steps, sync=False):
    n = c["tiles"] * c["width"]
    return _Tiled([dict(n=n, p=c["tiles"], order=c["order"], L=0 if sync else c["L"], nu=c["nu"],
                        dt=_dt(TWO_PI / n, c["nu"]), nsteps_max=steps, seed=seed,
                        dist=_dist(c["order"]),
                        cadv=0.8 if c.get("mode") == "linear" else None)])


def _exact_gradient(c, seed):
    n = c["tiles"] * c["width"]
    T = _tiled1d(c, seed, c["steps"])
    u, target = _field1d(n, seed), _field1d(n, seed + 1000003)
    h, seg = T.first(u), 10
    at_start = []
    for s in range(c["steps"]):
        if s % seg == 0:
            at_start.append((u, h))
        u, h = T.step(u, h, s)
    J, lam_u, lam_h = 0.5 * ((u - target) ** 2).sum(), u - target, torch.zeros_like(h)
    dnu = 0.0
    for i in reversed(range(len(at_start))):
        a, b = (x.detach().requires_grad_(True) for x in at_start[i])
        nu = torch.tensor(c["nu"], dtype=torch.float64, device="cuda", requires_grad=True)
        x, y = a, b
        for s in range(i * seg, min((i + 1) * seg, c["steps"])):
            x, y = T.step(x, y, s, nu)
        lam_u, lam_h, g = torch.autograd.grad((x, y), (a, b, nu), (lam_u, lam_h))
        dnu = dnu + g.cpu()
    return {"u": u, "J": J, "du0": lam_u, "dnu": dnu}


def _exact3d(c, seed):
    u = _field3d(c, seed)
    P, nn = (c["bx"], c["by"], c["bz"]), (c["nx"], c["ny"], c["nz"])
    W = tuple(n // p for n, p in zip(nn, P))
    kappa = torch.tensor([NU3] * 3 + list(_alpha(c)), dtype=torch.float64, device="cuda")
    kappa = kappa[:, None, None, None]
    dt = _dt3(c)
    nb = P[0] * P[1] * P[2]
    k_all = _delays(c["steps"], 6 * nb, c["L"], 2, UNIFORM, seed).reshape(-1, P[2], P[1], P[0], 6)
    depth = c["L"] + 2
    axis = {0: 3, 1: 2, 2: 1}                       # x, y, z in [c][z][y][x]
    hist = {(a, s): [] for a in range(3) for s in range(2)}

    def faces(v, a, s):
        """Edge planes of every block along axis a: its low (s=0) or high points."""
        return v.index_select(axis[a], torch.arange(P[a], device="cuda") * W[a] +
                              (W[a] - 1 if s else 0))

    def spread(k, a):
        """Block delays to the shape of the face planes along axis a."""
        for b, dim in ((2, 0), (1, 1), (0, 2)):
            if b != a:
                k = k.repeat_interleave(W[b], dim)
        return k[None]

    for n in range(c["steps"]):
        for key in hist:
            hist[key] = [faces(u, *key)] + hist[key][: depth - 1]
        lap = adv = None
        for a in range(3):
            dx = TWO_PI / nn[a]
            c1, c2 = 1.0 / (2.0 * dx), 1.0 / (dx * dx)
            side = []
            for s in range(2):
                v = torch.roll(u, -1 if s else 1, axis[a])
                k = spread(k_all[n, ..., 2 * a + s], a)
                # the facing plane of the neighbour block, by level
                lev = [torch.roll(x, -1 if s else 1, axis[a]) for x in hist[(a, 1 - s)]]
                hv = lev[0]
                for q in range(1, min(c["L"], len(lev) - 2) + 1):
                    hv = torch.where(k == q, lev[q] + float(q) * (lev[q] - lev[q + 1]), hv)
                v.index_copy_(axis[a], torch.arange(P[a], device="cuda") * W[a] +
                              (W[a] - 1 if s else 0), hv)
                side.append(v)
            lo, hi = side
            d2 = ((hi - 2.0 * u) + lo) * c2
            d1 = u[a] * ((hi - lo) * c1)
            lap = d2 if lap is None else lap + d2
            adv = d1 if adv is None else adv + d1
            del lo, hi, side, d1, d2
        u = u + dt * (kappa * lap - adv)
    return u


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "run3d":
        return _exact3d(c, seed)
    if kind == "gradient":
        return _exact_gradient(c, seed)
    if kind == "batch":
        ins = _instances(c, seed)
        T = _Tiled(ins)
        u = torch.cat([_field1d(i["n"], i["seed"], modes=6) for i in ins])
    else:
        # the weakly-synchronous run's delays are its own: the run without any
        # delay is its limit (the halo error is of the order of dt^2)
        steps = c["rounds"] * c["per_round"] if kind == "loop1d" else c["steps"]
        T = _tiled1d(c, seed, steps, sync=kind == "ws1d")
        u = _field1d(c["tiles"] * c["width"], seed)
    h = T.first(u)
    if kind == "loop1d":
        checks = []
        for s in range(c["rounds"] * c["per_round"]):
            u, h = T.step(u, h, s)
            if (s + 1) % c["per_round"] == 0:
                a = u.abs()
                checks.append(torch.stack([a.max(), u.mean(), a.sum(),
                                           (~torch.isfinite(u)).sum().double()]))
        return {"u": u, "checks": checks}
    for s in range(c["steps"]):
        u, h = T.step(u, h, s)
    return u
