"""What this framework is timed on: particle-in-cell steps through `PicSim` and `PicWindow`.

A case is a plain dict.  `kind` says how a program drives the simulation:

* ``step``       one fused step (`PicSim.step`), the loop of every production run;
* ``graph``      one replay of a captured HIP graph of `steps` steps, the launch-bound small batches;
* ``staged``     the rows of the time loop one call at a time, unfused, with the cell sort: programs that put
                 their own work between the rows, or want particles in cell order;
* ``monitored``  `steps` fused steps and the FP64 diagnostics (energies, Gauss and continuity residuals);
* ``window``     a differentiable window: forward with checkpoints, loss sum |E|^2, backward to the whole
                 initial state (`PicWindow`).

`profile` is the plasma: counter-streaming ``beams``, ``turbulence`` (guide field and random-phase modes),
``thermal`` boxes without fields, a pre-shocked ``shock`` between walls, a magnetised ``shear`` flow.  All
inputs are drawn on the GPU from the seed.  A simulation is advanced by every pass, as in a program's loop.
"""
from __future__ import annotations

import math
import random

import torch
from torch.utils.checkpoint import checkpoint

from paper_1906_06306_amd import _lib as L
from paper_1906_06306_amd.adjoint import PicWindow
from paper_1906_06306_amd.sim import Box, PicSim

COURANT = 0.45
SIDES = (64, 96, 128, 192, 256)      # of the batched boxes
PPCS = (4, 8, 16, 32)


def _case(name, **kw):
    base = dict(name=name, kind="step", profile="turbulence", dim=2, n0=256, n1=256, n2=1, t0=16, t1=16, t2=1,
                ppc=16, theta=0.3, precision="fp32", block=256, boxes=1, steps=1, capacity=8.0, walls=False,
                pusher="boris", filter_passes=0, fdtd_order=2, persistent=False)
    for k in kw:
        if k not in base:
            raise ValueError(k)
    return {**base, **kw}


def listed():
    return [
        # the smallest run: 65,536 particles in one dimension, FP64; every pass is launches and latency
        _case("two_stream_1d_fp64", profile="beams", dim=1, n0=512, n1=1, t0=8, t1=1, ppc=64, theta=0.01,
              precision="fp64", capacity=16.0),
        # a handful of small boxes advanced by graph replay, four steps at a time
        _case("graph_4_boxes_fp32", kind="graph", profile="thermal", boxes=4, steps=4, capacity=4.0),
        # a 2D run of ordinary size
        _case("turbulence_256_fp32"),
        # the largest 2D run: 33.5 million particles, the framework's headline workload
        _case("turbulence_1024_fp32", n0=1024, n1=1024),
        # the double-precision run that single precision is checked against
        _case("turbulence_512_fp64", n0=512, n1=512, precision="fp64", block=128),
        # parameter study: 64 independent boxes of uneven size, density and temperature in one batch
        _case("ensemble_64_fp32", profile="thermal", boxes=64, capacity=4.0),
        # 3D shock between conducting walls: 29 million particles, dense and thin tiles
        _case("shock_3d_fp32", profile="shock", dim=3, n0=256, n1=64, n2=64, t0=8, t1=8, t2=8, ppc=8, theta=3.286,
              block=512, walls=True, capacity=6.0),
        # a small periodic 3D box in double precision, sides that are no powers of two
        _case("box_3d_fp64", profile="thermal", dim=3, n0=64, n1=48, n2=40, t0=8, t1=8, t2=8, ppc=5,
              precision="fp64", capacity=4.0),
        # the alternative solvers (Higuera-Cary, eight binomial passes, fourth-order curls) on ragged tiles
        _case("solvers_ragged_fp32", n0=500, n1=336, t0=20, t1=12, ppc=7, pusher="hc", filter_passes=8,
              fdtd_order=4),
        # the rows of the loop called one by one, particles sorted by cell
        _case("staged_sorted_fp32", kind="staged", n0=512, n1=512),
        # a run that reads the FP64 diagnostics every five steps
        _case("monitored_512_fp32", kind="monitored", n0=512, n1=384, steps=5),
        # gradients through forty steps of a shear flow, checkpoints every eight steps
        _case("shear_window_fp32", kind="window", profile="shear", t0=8, t1=8, ppc=32, theta=0.1, steps=40,
              capacity=2.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["graph", "staged", "monitored", "window"])
    dim = 2 if kind == "window" else rng.choice([1, 2, 2, 2, 3, 3])
    precision = rng.choice(["fp32", "fp32", "fp64"])
    c = _case("", kind=kind, dim=dim, precision=precision, n1=1, t1=1)
    del c["name"]
    c["theta"] = round(_log(rng, 0.01, 1.0), 4)
    c["ppc"] = round(_log(rng, 3, 40))
    if dim == 1:
        c["t0"] = rng.choice([8, 10, 16, 32])
        c["n0"] = c["t0"] * round(_log(rng, 4, 1000))
        c["profile"], c["capacity"] = "beams", 16.0
    elif dim == 2:
        edges = [8, 16] if kind == "window" else [8, 12, 16, 16, 20, 32 if precision == "fp32" else 16]
        c["t0"] = rng.choice(edges)
        c["t1"] = c["t0"] if rng.random() < 0.7 else rng.choice(edges)
        cells = _log(rng, 1 << 11, 1 << (15 if kind == "window" else 19))
        aspect = _log(rng, 0.5, 2.0)
        c["n0"] = c["t0"] * max(3, round(math.sqrt(cells * aspect) / c["t0"]))
        c["n1"] = c["t1"] * max(3, round(math.sqrt(cells / aspect) / c["t1"]))
        c["profile"] = "shear" if kind == "window" else rng.choice(["turbulence", "turbulence", "thermal"])
        if c["profile"] == "thermal":
            c["boxes"], c["t0"], c["t1"], c["capacity"] = round(_log(rng, 2, 40)), 16, 16, 4.0
            c["n0"] = c["n1"] = 256
    else:
        c["t0"] = c["t1"] = c["t2"] = 8
        cells = _log(rng, 1 << 13, 1 << 18)
        for d in ("n0", "n1", "n2"):
            c[d] = 8 * max(3, round(cells ** (1 / 3) * rng.uniform(0.7, 1.4) / 8))
        c["ppc"] = min(c["ppc"], 16)
        c["walls"] = kind == "step" and rng.random() < 0.5
        c["profile"], c["capacity"] = ("shock" if c["walls"] else "thermal"), (8.0 if c["walls"] else 4.0)
        c["theta"] = 3.286 if c["walls"] else c["theta"]
    if kind == "graph":
        c["steps"] = rng.choice([1, 2, 4, 8])
    elif kind == "monitored":
        c["steps"] = rng.choice([1, 5, 10])
    elif kind == "window":
        c["steps"], c["capacity"] = rng.choice([8, 16, 24]), 3.0
    if kind in ("step", "graph"):
        c["block"] = rng.choice([128, 256, 256, 512])
        c["persistent"] = rng.random() < 0.15
        if rng.random() < 0.3:
            c["pusher"] = rng.choice(["vay", "hc"])
            if not c["walls"]:
                c["filter_passes"] = rng.choice([0, 1, 4, 8])
                c["fdtd_order"] = rng.choice([2, 4])
    return c


# ------------------------------------------------------------------- inputs


def _mean_gamma(theta):
    """Mean Lorentz factor of a Maxwell-Juttner distribution, by quadrature."""
    p = torch.linspace(0, 40.0 * max(theta, math.sqrt(theta)), 40001, dtype=torch.float64)
    g = torch.sqrt(1 + p * p)
    f = p * p * torch.exp((1 - g) / theta)
    return float((g * f).sum() / f.sum())


def _thermal_u(gen, theta, n, dev):
    """Isotropic Maxwell-Juttner four-velocities: |u| from its tabulated distribution function."""
    p = torch.linspace(0, 40.0 * max(theta, math.sqrt(theta)), 40001, dtype=torch.float64, device=dev)
    f = p * p * torch.exp((1 - torch.sqrt(1 + p * p)) / theta)
    cdf = torch.cumsum(f, 0)
    cdf = cdf / cdf[-1]
    r = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    i = torch.searchsorted(cdf, r).clamp_(1, p.numel() - 1)
    a, b = cdf[i - 1], cdf[i]
    mag = p[i - 1] + (p[i] - p[i - 1]) * ((r - a) / (b - a).clamp_min(1e-300))
    mu = 2 * torch.rand(n, generator=gen, device=dev, dtype=torch.float64) - 1
    phi = 2 * math.pi * torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    st = torch.sqrt(1 - mu * mu)
    return torch.stack([mag * st * torch.cos(phi), mag * st * torch.sin(phi), mag * mu])


def _boosted(u, gamma_b, sign):
    beta = sign * math.sqrt(1 - 1 / gamma_b ** 2)
    g = torch.sqrt(1 + (u * u).sum(0))
    return torch.cat([(gamma_b * (u[0] + beta * g))[None], u[1:]])


def _quiet(gen, dim, n, ppc, dev, x0=0):
    """ppc particles in every cell, layer by layer, uniform inside the cell."""
    N = n[0] * n[1] * n[2]
    k = torch.arange(N, device=dev)
    idx = (k % n[0] + x0, (k // n[0]) % n[1], k // (n[0] * n[1]))
    return torch.stack([(idx[d] + torch.rand((ppc, N), generator=gen, device=dev, dtype=torch.float64)).reshape(-1)
                        for d in range(dim)])


def _box(case, n, ppc, theta, gen, dev):
    """One box in code units: cells of size 1, skin depth of a few cells."""
    D, profile = case["dim"], case["profile"]
    N = n[0] * n[1] * n[2]
    E = torch.zeros((3, N), dtype=torch.float64, device=dev)
    B = torch.zeros((3, N), dtype=torch.float64, device=dev)
    skin, gam = 3.0, _mean_gamma(theta)
    if profile == "shock":
        # a quarter of the box hot and four times as dense, the rest a cold beam towards the wall at x = 0
        xs = n[0] // 4
        x = torch.cat([_quiet(gen, D, (xs, n[1], n[2]), 4 * ppc, dev),
                       _quiet(gen, D, (n[0] - xs, n[1], n[2]), ppc, dev, xs)], 1)
        nd = 4 * ppc * xs * n[1] * n[2]
        us = [torch.cat([_thermal_u(gen, theta, nd, dev),
                         _boosted(_thermal_u(gen, 1e-4, x.shape[1] - nd, dev), 10.0, -1.0)], 1) for _ in range(2)]
        skin, gam = 10.0, 10.0
    else:
        x = _quiet(gen, D, n, ppc, dev)
        us = [_thermal_u(gen, theta, x.shape[1], dev) for _ in range(2)]
        if profile == "beams":
            half = x.shape[1] // 2
            us = [torch.cat([_boosted(u[:, :half], 3.0, 1.0), _boosted(u[:, half:], 3.0, -1.0)], 1) for u in us]
            skin, gam = 10.0, 3.0 * gam
    q = (COURANT / skin) ** 2 * gam / (2 * ppc)
    if profile in ("turbulence", "shear"):
        sigma = 10.0 if profile == "turbulence" else 1.0
        B0 = math.sqrt(sigma * ppc * q * COURANT ** 2 * gam * 2)
        B[2] = B0
    if profile == "turbulence" and D == 2:
        ph = 2 * math.pi * torch.rand((2, 8, 8), generator=gen, device=dev, dtype=torch.float64)
        m = torch.arange(1, 9, device=dev, dtype=torch.float64)
        amp = 2 * B0 / (8 * torch.sqrt(m[:, None] ** 2 + m[None, :] ** 2)) * (n[0] / (2 * math.pi))
        A = torch.zeros((n[1], n[0]), dtype=torch.float64, device=dev)
        ys, xs = (torch.arange(v, device=dev, dtype=torch.float64) * (2 * math.pi / v) for v in (n[1], n[0]))
        for i in range(8):
            for j in range(8):
                A += amp[i, j] * torch.sin(m[j] * ys + ph[1, i, j])[:, None] * torch.sin(m[i] * xs + ph[0, i, j])
        B[0] = (torch.roll(A, -1, 0) - A).reshape(-1)
        B[1] = -(torch.roll(A, -1, 1) - A).reshape(-1)
    if profile == "shear":
        for u in us:
            u[0] += 0.1 * torch.sin(2 * math.pi * x[1] / n[1])
    return Box(D=D, n=n, c=COURANT, charge=[-q, q], qm=[-1.0, 1.0], mass=[q, q], pos=[x, x.clone()], u=us, E=E, B=B)


def _shapes(case):
    """(cells, particles per cell and species, temperature) of every box."""
    if case["boxes"] == 1:
        return [((case["n0"], case["n1"], case["n2"]), case["ppc"], case["theta"])]
    r = random.Random(case["boxes"])
    out = []
    for _ in range(case["boxes"]):
        n = (r.choice(SIDES), r.choice(SIDES), 1)
        out.append((n, r.choice(PPCS), round(10 ** r.uniform(-2, 0), 4)))
    return out


def _boxes(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    return [_box(case, n, ppc, theta, gen, dev) for n, ppc, theta in _shapes(case)]


def _tile(case):
    return (case["t0"], case["t1"], case["t2"])[:case["dim"]]


def _clear_free_slots(sim):
    """Free slots of the particle planes hold no particle; zero them, so that whole planes can be compared."""
    pos, u, _, off, cnt = sim.particle_views()
    off, cnt = off.reshape(-1), cnt.reshape(-1)
    cap = pos.shape[1]
    for a in range(0, cap, 1 << 25):
        k = torch.arange(a, min(cap, a + (1 << 25)), device=pos.device)
        seg = torch.searchsorted(off, k, right=True) - 1
        free = k - off[seg] >= cnt[seg]
        for plane in (*pos, *u):
            plane[a:a + k.numel()].masked_fill_(free, 0)


def prepare(case, seed):
    boxes = _boxes(case, seed)
    if case["kind"] == "window":
        b = boxes[0]
        settings = dict(D=b.D, n=b.n, c=b.c, charge=b.charge, qm=b.qm, mass=b.mass, nsteps=case["steps"], window=8,
                        precision=case["precision"], tile=_tile(case), capacity_factor=case["capacity"])
        return dict(kind="window", settings=settings,
                    leaves=[b.E, b.B, *(t for k in range(2) for t in (b.pos[k], b.u[k]))])
    torch.cuda.synchronize()
    sim = PicSim(boxes, tile=_tile(case), precision=case["precision"], block=case["block"],
                 capacity_factor=case["capacity"], walls=case["walls"], pusher=case["pusher"],
                 filter_passes=case["filter_passes"], fdtd_order=case["fdtd_order"],
                 options=L.PIC_OPT_PERSISTENT if case["persistent"] else 0,
                 stream=torch.cuda.Stream() if case["kind"] == "graph" else None)
    torch.cuda.synchronize()
    _clear_free_slots(sim)
    torch.cuda.synchronize()
    if case["kind"] == "graph":
        sim.capture(case["steps"])
    pos, u, _, _, cnt = sim.particle_views()
    return dict(kind=case["kind"], sim=sim, steps=case["steps"], state=[*sim.field_views(), pos, u, cnt])


def run(state):
    kind = state["kind"]
    if kind == "window":
        leaves = [t.detach().requires_grad_() for t in state["leaves"]]
        E, B = PicWindow.apply(state["settings"], *leaves)
        (E * E).sum().backward()
        return [E.detach(), B.detach(), *(t.grad for t in leaves)]
    sim = state["sim"]
    if kind == "step":
        sim.step(state["steps"], half_b_in_push=True)
    elif kind == "graph":
        sim.replay(1)
    elif kind == "staged":
        sim.fdtd(L.PIC_HALF_B)
        sim.push(fused=False)
        sim.fdtd(L.PIC_HALF_B)
        sim.deposit()
        sim.fdtd(L.PIC_CURL_E_ADD_J)
        sim.sort_migrate(sort_cells=True)
    else:
        sim.step(state["steps"], half_b_in_push=True)
        d = sim.diagnostics()
        out = [*state["state"], d["field_energy"], d["kinetic_energy"], d["particles"], d["near_face"]]
        if sim.prec == L.PIC_FP32:
            # residuals: rounding noise of the state's precision, of which only the leading figures mean anything
            out.append(torch.tensor([d["gauss_max"], d["divb_max"]], dtype=torch.float32))
        return out
    return state["state"]


# --------------------------------------------------------------------- work


def work(case):
    D, w = case["dim"], (8 if case["precision"] == "fp64" else 4)
    np_, nc = 0, 0
    for n, ppc, _ in _shapes(case):
        cells = n[0] * n[1] * n[2]
        nc += cells
        layers = 4 * ppc * (n[0] // 4) + ppc * (n[0] - n[0] // 4) if case["profile"] == "shock" else ppc * n[0]
        np_ += 2 * layers * n[1] * n[2]
    # a step reads and writes every particle and E, B, J of every cell once
    push = 6 * 3 * (2 ** D - 1) + 80 + (40, 70, 130)[D - 1]
    step_bytes = np_ * 2 * (D + 3) * w + nc * 18 * w
    step_flops = np_ * push + nc * 40
    k = case["steps"]
    if case["kind"] == "window":
        # forward, and a reverse sweep that reads the state and the adjoints and writes the adjoints
        return dict(bytes=k * (step_bytes + np_ * 3 * (D + 3) * w + nc * 18 * w), flops=4 * k * step_flops)
    out = dict(bytes=k * step_bytes, flops=k * step_flops)
    if case["kind"] == "monitored":
        out["bytes"] += np_ * (D + 3) * w + nc * 9 * w
        out["flops"] += np_ * 40
    return out


# ------------------------------------------- the same step in plain 64 bits


def _diff(F, axis, sign, D, order):
    """Forward (sign = 1) or backward difference along grid axis 0..2 (x is the last storage axis)."""
    if axis >= D:
        return torch.zeros_like(F)
    ax = F.dim() - 1 - axis

    def at(o):
        return torch.roll(F, -o, ax)

    if sign > 0:
        near, far = at(1) - F, (at(2) - at(-1) if order == 4 else None)
    else:
        near, far = F - at(-1), (at(1) - at(-2) if order == 4 else None)
    return 9 / 8 * near - 1 / 24 * far if order == 4 else near


def _curl(F, sign, D, order):
    d = lambda m, a: _diff(F[m], a, sign, D, order)  # noqa: E731
    return torch.stack([d(2, 1) - d(1, 2), d(0, 2) - d(2, 0), d(1, 0) - d(0, 1)])


def _gather(F, half, x, n, D, walls):
    """Linear interpolation of one component from its own staggered lattice."""
    flat, corners = F.reshape(-1), [(0, 1.0)]
    stride = 1
    for d in range(D):
        s = x[d] - (0.5 if half[d] else 0.0)
        i = torch.floor(s).detach()
        w = s - i
        i = i.long()
        new = []
        for o, wt in ((0, 1 - w), (1, w)):
            j = i + o
            if d == 0 and walls and half[0]:
                j = j.clamp(0, n[0] - 1)         # the wall is a mirror
            j = torch.remainder(j, n[d]) * stride
            new += [(idx + j, wgt * wt) for idx, wgt in corners]
        corners = new
        stride *= n[d]
    return sum(flat[idx] * wgt for idx, wgt in corners)


def _rotate(w, t):
    wt = (w * t).sum(0)
    return (w + wt * t + torch.linalg.cross(w, t, dim=0)) / (1 + (t * t).sum(0))


def _kick(u, e, b, c, s, pusher):
    k = 0.5 * s / c

    def implicit(w, tau):
        sg = 1 + (w * w).sum(0) / c ** 2 - (tau * tau).sum(0)
        us = (w * tau).sum(0) / c
        return torch.sqrt(0.5 * (sg + torch.sqrt(sg * sg + 4 * ((tau * tau).sum(0) + us * us))))

    if pusher == "vay":
        v = c * u / torch.sqrt(1 + (u * u).sum(0))
        w = c * u + s * e + torch.linalg.cross(v, k * b, dim=0)
        return _rotate(w, k * b / implicit(w, k * b)) / c
    eps = 0.5 * s * e
    w = c * u + eps
    if pusher == "hc":
        t = k * b / implicit(w, k * b)
        w = _rotate(w, t)
        return (w + eps + torch.linalg.cross(w, t, dim=0)) / c
    t = k * b / torch.sqrt(1 + (w * w).sum(0) / c ** 2)
    u2 = 2 / (1 + (t * t).sum(0)) * (w + torch.linalg.cross(w, t, dim=0))
    return (w + torch.linalg.cross(u2, t, dim=0) + eps) / c


def _zigzag(J, x1, x2, dv, q, n, D):
    """Adds the ZigZag current of moves x1 -> x2 to the flat planes J."""
    segs = [[], []]
    for d in range(3):
        if d < D:
            a, b = x1[d], x2[d]
            fa, fb = torch.floor(a).detach(), torch.floor(b).detach()
            xr = torch.minimum(torch.minimum(fa, fb) + 1, torch.maximum(torch.maximum(fa, fb), 0.5 * (a + b)))
            segs[0].append((xr - a, 0.5 * (a + xr) - fa, fa.long()))
            segs[1].append((b - xr, 0.5 * (b + xr) - fb, fb.long()))
        else:
            for sg in segs:
                sg.append((0.5 * dv[d], None, None))
    stride = (1, n[0], n[0] * n[1])
    for sg in segs:
        for m in range(3):
            trans = [d for d in range(D) if d != m]
            parts = [(0, 1.0)]
            for d in trans:
                _, w, i = sg[d]
                parts = [(idx + torch.remainder(i + o, n[d]) * stride[d], wt * ((1 - w) if o == 0 else w))
                         for idx, wt in parts for o in (0, 1)]
            if len(trans) == 2:
                cr = sg[trans[0]][0] * sg[trans[1]][0] / 12
                parts = [(idx, wt + (cr if k in (0, 3) else -cr)) for k, (idx, wt) in enumerate(parts)]
            base = torch.remainder(sg[m][2], n[m]) * stride[m] if m < D else 0
            for idx, wt in parts:
                J[m] = J[m].index_add(0, base + idx, q * sg[m][0] * wt) if J[m].requires_grad or dv.requires_grad \
                    else J[m].index_add_(0, base + idx, q * sg[m][0] * wt)


def _move(J, E, B, x, u, q, s, c, n, D, walls, pusher):
    """Push of one species and its current."""
    halves = [[d == m for d in range(3)] for m in range(3)] + [[d != m for d in range(3)] for m in range(3)]
    f = [_gather((E[m] if m < 3 else B[m - 3]), halves[m], x, n, D, walls) for m in range(6)]
    u = _kick(u, torch.stack(f[:3]), torch.stack(f[3:]), c, s, pusher)
    dv = c * u / torch.sqrt(1 + (u * u).sum(0))
    x2 = x + dv[:D]
    if walls:
        out = (x2[0] < 0) | (x2[0] >= n[0])
        wall = torch.where(x2[0] < 0, 0.0, float(n[0]))
        t = torch.where(out, (wall - x[0]) / torch.where(out, x2[0] - x[0], 1.0), 1.0)
        i = out.nonzero().squeeze(1)
        # the broken path: to the wall, and from there to the mirrored end
        at_wall = x[:, i] + t[i] * (x2[:, i] - x[:, i])
        at_wall[0] = wall[i]
        end = x2[:, i].clone()
        end[0] = (2 * wall[i] - end[0]).clamp_max(math.nextafter(n[0], 0.0))
        keep = (~out).nonzero().squeeze(1)
        _zigzag(J, x[:, keep], x2[:, keep], dv[:, keep], q, n, D)
        _zigzag(J, x[:, i], at_wall, dv[:, i] * t[i], q, n, D)
        _zigzag(J, at_wall, end, dv[:, i] * (1 - t[i]), q, n, D)
        x2 = x2.index_copy(1, i, end)
        u = u.clone()
        u[0, i] = -u[0, i]
    else:
        _zigzag(J, x, x2, dv, q, n, D)
    n_ = torch.tensor(n[:D], dtype=x.dtype, device=x.device)[:, None]
    return x2 - torch.floor(x2 / n_).detach() * n_, u


def _step64(case, box, E, B, parts, chunk=1 << 22):
    """One whole step; E, B as (3, n2, n1, n0), parts as [(x, u) per species]."""
    n, D, c, order = box.n, box.D, box.c, case["fdtd_order"]
    h = 0.5 * c * _curl(E, 1, D, order)
    Bn = B - h
    J = [torch.zeros(E[0].numel(), dtype=E.dtype, device=E.device) for _ in range(3)]
    out = []
    for k, (x, u) in enumerate(parts):
        if x.requires_grad or E.requires_grad:
            out.append(_move(J, E, Bn, x, u, box.charge[k], box.qm[k], c, n, D, case["walls"], case["pusher"]))
            continue
        xs, us = torch.empty_like(x), torch.empty_like(u)
        for a in range(0, x.shape[1], chunk):
            xs[:, a:a + chunk], us[:, a:a + chunk] = _move(J, E, Bn, x[:, a:a + chunk], u[:, a:a + chunk],
                                                           box.charge[k], box.qm[k], c, n, D, case["walls"],
                                                           case["pusher"])
        out.append((xs, us))
    Bn = Bn - h
    J = torch.stack(J).reshape(E.shape)
    for _ in range(case["filter_passes"]):
        for d in range(D):
            ax = J.dim() - 1 - d
            J = 0.25 * torch.roll(J, 1, ax) + 0.5 * J + 0.25 * torch.roll(J, -1, ax)
    E = E + c * _curl(Bn, -1, D, order) - J
    if case["walls"]:
        E[1:, ..., 0] = 0
    return E, Bn, J, out


def exact(case, seed):
    k = case["steps"] + (1 if case["kind"] == "graph" else 0)      # capturing runs one step
    boxes = _boxes(case, seed)
    if case["kind"] == "window":
        b = boxes[0]
        shape = (3, b.n[2], b.n[1], b.n[0])
        leaves = [t.requires_grad_() for t in (b.E, b.B, b.pos[0], b.u[0], b.pos[1], b.u[1])]

        def one(E, B, xe, ue, xp, up):
            E, B, _, parts = _step64(case, b, E, B, [(xe, ue), (xp, up)])
            return (E, B, *parts[0], *parts[1])

        st = (leaves[0].reshape(shape), leaves[1].reshape(shape), *leaves[2:])
        for _ in range(k):
            st = checkpoint(one, *st, use_reentrant=False)
        (st[0] * st[0]).sum().backward()
        return [st[0].detach().reshape(3, -1), st[1].detach().reshape(3, -1), *(t.grad for t in leaves)]
    fields = [], [], []
    for b in boxes:
        shape = (3, b.n[2], b.n[1], b.n[0])
        E, B = b.E.reshape(shape), b.B.reshape(shape)
        parts = [(b.pos[s], b.u[s]) for s in range(2)]
        for _ in range(k):
            E, B, J, parts = _step64(case, b, E, B, parts)
        for f, v in zip(fields, (E, B, J)):
            f.append(v.reshape(3, -1))
    E, B, J = (torch.cat(f, 1) for f in fields)
    # positions and momenta are stored by tile, in the order of the moves between tiles: held to the bits of
    # their own type, not to these global coordinates
    out = [E, B, J, None, None, None]
    if case["kind"] == "monitored":
        kin = sum(m * b.c ** 2 * float((torch.sqrt(1 + (u * u).sum(0)) - 1).sum())
                  for (_, u), m in zip(parts, boxes[0].mass))
        out += [0.5 * float((E * E + B * B).sum()), kin, None, None]
    return out
