"""Workloads by which the speed of this framework is followed, through its public
entry points.  Each case is a dict of plain values; ``prepare`` makes what a user's
program holds before the call (inputs drawn on the device from the seed, and the
context that such a program keeps), ``run`` is one pass, ``work`` what the pass
cannot do without and ``exact`` the direct sum in float64.

Kinds of pass:

* ``static``   bh_forces_static: one small system without device allocation;
* ``forces``   build_tree + compute_forces of a system not seen before;
* ``restart``  set_state + compute_forces + batch_run in a kept context: one short
               integration from given initial conditions (replayed graphs);
* ``steps``    leapfrog_step in a running integration, then the state and energy;
* ``batch``    batch_run of many uneven clusters in a running integration;
* ``load``     batch_build + batch_forces of clusters with settings of their own;
* ``active``   refit + compute_forces_active: the inner operation of a caller that
               drives individual time-steps;
* ``block``    block_step in a running integration;
* ``serve``    a server that takes a handful of requests and runs until all are done.
"""

import math

import numpy as np
import torch

import paper_1106_1900_amd as bh

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # the smallest call: one force evaluation of a small system from a loop
        # that may not allocate; latency and launches are all it is
        dict(name="static_1500", kind="static", model="plummer", n=1500, theta=0.75, eps=0.02),
        # the small system of the benchmark, loaded and evaluated once
        dict(name="forces_4k", kind="forces", model="plummer", n=4096, theta=0.5, eps=0.01,
             mac=0, nleaf=16, ncrit=64),
        # the same system integrated for a few steps from new initial conditions
        dict(name="restart_4k", kind="restart", model="plummer", n=4096, theta=0.5, eps=0.01,
             dt=1.0 / 512, steps=4),
        # an ordinary single snapshot, odd size, cuspy, the other opening test
        dict(name="forces_100k_min", kind="forces", model="hernquist", n=100003, theta=0.6,
             eps=0.02, mac=1, nleaf=16, ncrit=64),
        # the encounter of two galaxies with black holes, step by step
        dict(name="merger_240k", kind="steps", model="merger", n=240002, theta=0.75, eps=0.1,
             dt=1.0 / 64, steps=2),
        # the headline: steps of a Plummer sphere of 2^20 particles
        dict(name="steps_1m", kind="steps", model="plummer", n=1 << 20, theta=0.75, eps=1.0 / 64,
             dt=1.0 / 512, steps=2),
        # refit and the walk of the groups that hold 1% active particles
        dict(name="active_1m", kind="active", model="plummer", n=1 << 20, theta=0.75,
             eps=1.0 / 64, share=0.01),
        # the large galaxy at a small opening angle
        dict(name="galaxy_4m", kind="steps", model="galaxy", n=1 << 22, theta=0.4, eps=0.02,
             dt=1.0 / 128, steps=1),
        # many uneven clusters advanced together, one replayed step
        dict(name="batch_512", kind="batch", k=512, nmin=1024, nmax=65536, theta=0.75,
             dt=1.0 / 512, steps=1),
        # a few small clusters with settings of their own, loaded and evaluated
        dict(name="load_24", kind="load", k=24, nmin=300, nmax=20000),
        # block time-steps of a system with a wide range of accelerations
        dict(name="block_130k", kind="block", model="hernquist", n=130007, theta=0.75, eps=0.02,
             dt=1.0 / 128, eta=0.0003, level=4, growth=0.1),
        # the serving loop with a mixed handful of requests
        dict(name="serve_20", kind="serve", k=20, nmin=1024, nmax=65536, steps=2, dt=1.0 / 256),
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["static", "forces", "forces", "restart", "steps", "steps", "active",
                       "batch", "load", "block", "serve"])
    theta = rng.choice([0.4, 0.5, 0.6, 0.75])
    eps = rng.choice([0.005, 0.01, 1.0 / 64, 0.02, 0.05])
    model = rng.choice(["plummer", "hernquist", "galaxy"])
    if kind == "static":
        return dict(kind=kind, model=model, n=_log_int(rng, 200, 32768), theta=theta, eps=eps)
    if kind == "forces":
        return dict(kind=kind, model=model, n=_log_int(rng, 1000, 1500000), theta=theta, eps=eps,
                    mac=rng.choice([0, 0, 1]), nleaf=rng.choice([16, 16, 8, 32]),
                    ncrit=rng.choice([64, 64, 32, 128]))
    if kind == "restart":
        return dict(kind=kind, model=model, n=_log_int(rng, 1000, 200000), theta=theta, eps=eps,
                    dt=1.0 / 512, steps=rng.choice([2, 4]))
    if kind == "steps":
        return dict(kind=kind, model=model, n=_log_int(rng, 3000, 2500000), theta=theta, eps=eps,
                    dt=1.0 / 256, steps=1)
    if kind == "active":
        return dict(kind=kind, model=model, n=_log_int(rng, 20000, 1500000), theta=theta, eps=eps,
                    share=rng.choice([0.001, 0.01, 0.1]))
    if kind == "batch":
        return dict(kind=kind, k=_log_int(rng, 8, 300), nmin=1024, nmax=65536, theta=theta,
                    dt=1.0 / 512, steps=1)
    if kind == "load":
        return dict(kind=kind, k=_log_int(rng, 4, 100), nmin=_log_int(rng, 100, 1000), nmax=20000)
    if kind == "block":
        return dict(kind=kind, model=rng.choice(["plummer", "hernquist"]),
                    n=_log_int(rng, 10000, 300000), theta=theta, eps=0.02, dt=1.0 / 128, eta=0.0003,
                    level=rng.choice([2, 3, 4]), growth=0.1)
    return dict(kind=kind, k=_log_int(rng, 4, 40), nmin=1024, nmax=65536, steps=2, dt=1.0 / 256)


# ---------------------------------------------------------------------------
# inputs: model systems drawn on the device (G = 1, total mass 1, at rest)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _u(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=F64)


def _iso(g, n):
    c = 2.0 * _u(g, n) - 1.0
    p = 2.0 * math.pi * _u(g, n)
    s = torch.sqrt((1.0 - c * c).clamp_min(0.0))
    return torch.stack([s * torch.cos(p), s * torch.sin(p), c], 1)


def _table(x, xp, fp):
    """Linear interpolation in an ascending table (numpy arrays xp, fp)."""
    xp = torch.as_tensor(xp, device=DEV, dtype=F64)
    fp = torch.as_tensor(fp, device=DEV, dtype=F64)
    i = torch.searchsorted(xp, x).clamp(1, xp.numel() - 1)
    w = (x - xp[i - 1]) / (xp[i] - xp[i - 1])
    return fp[i - 1] + w.clamp(0.0, 1.0) * (fp[i] - fp[i - 1])


def _plummer(g, n):
    r = 1.0 / torch.sqrt((0.999 * _u(g, n)).clamp_min(1e-12) ** (-2.0 / 3.0) - 1.0)
    q = np.linspace(0.0, 1.0, 2049)
    f = q * q * (1.0 - q * q) ** 3.5
    cdf = np.concatenate([[0.0], np.cumsum(0.5 * (f[1:] + f[:-1]))])
    v = _table(_u(g, n), cdf / cdf[-1] + 1e-15 * np.arange(2049), q)
    v = v * math.sqrt(2.0) * (1.0 + r * r) ** -0.25
    pos = r[:, None] * _iso(g, n) * (3.0 * math.pi / 16.0)
    vel = v[:, None] * _iso(g, n) * math.sqrt(16.0 / (3.0 * math.pi))
    return pos, vel, torch.full((n,), 1.0 / n, device=DEV, dtype=F64)


def _hernquist(g, n):
    s = torch.sqrt(0.99 * _u(g, n))
    r = s / (1.0 - s)
    grid = np.geomspace(1e-5, 1e4, 3000)
    f = 1.0 / (2.0 * np.pi) / (grid * (grid + 1.0) ** 5)          # rho M / r^2
    seg = 0.5 * (f[1:] + f[:-1]) * np.diff(grid)
    tail = np.concatenate([np.cumsum(seg[::-1])[::-1], [0.0]])
    sig = np.sqrt(tail * 2.0 * np.pi * grid * (grid + 1.0) ** 3)
    vel = _table(r, grid, sig)[:, None] * torch.randn(n, 3, generator=g, device=DEV, dtype=F64)
    return r[:, None] * _iso(g, n), vel, torch.full((n,), 1.0 / n, device=DEV, dtype=F64)


def _galaxy(g, n):
    """Exponential disk, Hernquist bulge and truncated NFW halo: a quarter, an
    eighth and the rest of the particles, masses 1 : 0.3 : 10."""
    nd, nb = n // 4, n // 8
    nh = n - nd - nb
    x = np.linspace(0.0, 60.0, 6001)
    R = _table(_u(g, nd) * (1.0 - 1e-9), 1.0 - (1.0 + x) * np.exp(-x) + 1e-15 * np.arange(6001), x)
    z = 0.1 * torch.atanh((2.0 * _u(g, nd) - 1.0).clamp(-1 + 1e-9, 1 - 1e-9))
    ph = 2.0 * math.pi * _u(g, nd)
    pd = torch.stack([R * torch.cos(ph), R * torch.sin(ph), z], 1)
    s = torch.sqrt(0.99 * _u(g, nb))
    rb = 0.2 * s / (1.0 - s)
    y = np.linspace(0.0, 10.0, 8001)
    rh = 2.0 * _table(_u(g, nh), (np.log1p(y) - y / (1.0 + y)) / (math.log(11.0) - 10.0 / 11.0), y)
    md, mb, mh = 1.0 / 11.3, 0.3 / 11.3, 10.0 / 11.3

    def vc2(r):         # squared circular speed of the enclosed mass
        q = (r / 2.0).clamp_max(10.0)
        m = md * (1.0 - (1.0 + r) * torch.exp(-r)) + mb * r * r / (r + 0.2) ** 2
        return (m + mh * (torch.log1p(q) - q / (1.0 + q)) / (math.log(11.0) - 10.0 / 11.0)) / r.clamp_min(1e-3)

    def normal(k):
        return torch.randn(k, 3, generator=g, device=DEV, dtype=F64)

    vc = torch.sqrt(vc2(R))
    vd = torch.stack([-vc * torch.sin(ph), vc * torch.cos(ph), 0.0 * vc], 1) + 0.1 * vc[:, None] * normal(nd)
    vs = [0.6 * torch.sqrt(vc2(r))[:, None] * normal(r.numel()) for r in (rb, rh)]
    pos = torch.cat([pd, rb[:, None] * _iso(g, nb), rh[:, None] * _iso(g, nh)])
    mass = torch.cat([torch.full((k,), m / max(k, 1), device=DEV, dtype=F64)
                      for k, m in ((nd, md), (nb, mb), (nh, mh))])
    return pos, torch.cat([vd] + vs), mass


def _merger(g, n):
    """Two galaxies, masses 1 : 1/3, each with a black hole of 0.1% of its mass at
    its centre, 40 apart on a parabolic orbit with pericentre 4."""
    parts, left = [], n
    for m in (1.0, 1.0 / 3.0):
        k = left if m < 1.0 else n // 2
        left -= k
        p, v, w = _galaxy(g, k - 1)
        s = m ** (1.0 / 3.0)
        zero = torch.zeros(1, 3, device=DEV, dtype=F64)
        parts.append((torch.cat([p * s, zero]), torch.cat([v * s, zero]),
                      torch.cat([w * m, torch.full((1,), 1e-3 * m, device=DEV, dtype=F64)])))
    M, d, rp = 1.001 * 4.0 / 3.0, 40.0, 4.0
    vt = math.sqrt(2.0 * M * rp) / d
    at = torch.tensor([d, 0.0, 0.0], device=DEV, dtype=F64)
    u = torch.tensor([-math.sqrt(2.0 * M / d - vt * vt), vt, 0.0], device=DEV, dtype=F64)
    a, b = parts
    return (torch.cat([a[0] - 0.25 * at, b[0] + 0.75 * at]),
            torch.cat([a[1] - 0.25 * u, b[1] + 0.75 * u]), torch.cat([a[2], b[2]]))


_MODELS = dict(plummer=_plummer, hernquist=_hernquist, galaxy=_galaxy, merger=_merger)


def _system(model, n, seed):
    pos, vel, mass = _MODELS[model](_gen(seed), n)
    m = mass[:, None] / mass.sum()
    return ((pos - (m * pos).sum(0)).contiguous(), (vel - (m * vel).sum(0)).contiguous(),
            mass.contiguous())


def _table_of(case):
    """Sizes (log-uniform) and settings of a batch's or a trace's systems.  They
    belong to the case and are the same for every seed."""
    rng = np.random.default_rng([case["k"], case["nmin"], case["nmax"]])
    tab = []
    for _ in range(case["k"]):
        n = int(math.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]))))
        q = dict(n=n, theta=float(rng.choice([0.5, 0.75])), eps=float(rng.choice([0.01, 0.02])),
                 dt=case.get("dt", 0.0))
        own = dict(mac=int(rng.integers(0, 4) == 0), nleaf=int(rng.choice([8, 16, 16, 32])),
                   ncrit=int(rng.choice([32, 64, 64, 128])))
        q["model"] = str(rng.choice(["plummer", "hernquist"]))
        if case["kind"] == "batch":
            q.update(theta=case["theta"], eps=0.04 * n ** (-1.0 / 3.0), model="plummer")
        if case["kind"] == "load":
            q.update(own)
        tab.append(q)
    return tab


def _clusters(case, seed):
    tab = _table_of(case)
    return tab, [_system(q["model"], q["n"], 1000003 * int(seed) + i) for i, q in enumerate(tab)]


# ---------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("batch", "load", "serve"):
        s["table"], sys = _clusters(case, seed)
        if kind == "serve":
            s["systems"] = sys
            s["srv"] = bh.Server(hbm_budget_bytes=4 << 30, max_requests=64)
            return s
        s["pos"], s["vel"], s["mass"] = (torch.cat([q[j] for q in sys]).contiguous() for j in range(3))
        s["ctx"] = ctx = bh.Context()
        if kind == "batch":
            ctx.batch_build(s["table"], s["pos"], s["mass"], s["vel"])
            ctx.batch_forces(want=False)
        return s
    s["pos"], s["vel"], s["mass"] = pos, vel, mass = _system(case["model"], case["n"], seed)
    if kind == "static":
        return s
    s["ctx"] = ctx = bh.Context(nleaf=case.get("nleaf", 16), ncrit=case.get("ncrit", 64))
    if kind == "forces":
        ctx.set_mac(case["mac"])
        return s
    ctx.build_tree(pos, mass)
    ctx.set_velocities(vel)
    ctx.compute_forces(case["theta"], case["eps"], want=False)
    if kind == "restart":
        ctx.batch_set_params([_restart(case)])
    if kind == "active":
        s["mask"] = (torch.rand(case["n"], generator=_gen(seed + 1), device=DEV) < case["share"]).to(torch.uint8)
    return s


def _restart(case):
    return dict(n=case["n"], theta=case["theta"], eps=case["eps"], dt=case["dt"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "static":
        return bh.forces_static(s["pos"], s["mass"], case["theta"], case["eps"])
    if kind == "serve":
        return _serve(s)
    ctx = s["ctx"]
    if kind == "forces":
        ctx.build_tree(s["pos"], s["mass"])
        return ctx.compute_forces(case["theta"], case["eps"])
    if kind == "load":
        ctx.batch_build(s["table"], s["pos"], s["mass"], s["vel"])
        return ctx.batch_forces()
    if kind == "restart":
        ctx.set_state(s["pos"], s["vel"])
        ctx.compute_forces(case["theta"], case["eps"], want=False)
        ctx.batch_run(case["steps"])
        return ctx.get_state()
    if kind == "steps":
        for _ in range(case["steps"]):
            ctx.leapfrog_step(case["dt"])
        return ctx.get_state(), ctx.energy()[:3]
    if kind == "batch":
        ctx.batch_run(case["steps"])
        return ctx.get_state()
    if kind == "active":
        ctx.refit()
        return ctx.compute_forces_active(case["theta"], case["eps"], s["mask"])
    ctx.block_step(case["dt"], case["eta"], case["eps"], case["level"], case["growth"])
    return ctx.get_state()


def _serve(s):
    srv, out, tickets = s["srv"], [], []
    for q, (pos, vel, mass) in zip(s["table"], s["systems"]):
        o = (torch.empty_like(pos), torch.empty_like(vel),
             torch.empty(pos.shape, dtype=torch.float32, device=DEV),
             torch.empty(mass.shape, dtype=torch.float32, device=DEV))
        tickets.append(srv.submit(pos, mass, vel, theta=q["theta"], eps=q["eps"], dt=q["dt"],
                                  nsteps=s["case"]["steps"], out_pos=o[0], out_vel=o[1],
                                  out_acc=o[2], out_pot=o[3]))
        out.append(o)
    waiting = set(tickets)
    while waiting:
        srv.step()
        waiting = {t for t in waiting if srv.poll(t)["state"] < bh.REQ_DONE}
    for t in tickets:
        srv.release(t)
    return [torch.cat([o[j] for o in out]) for j in range(4)]


# ---------------------------------------------------------------------------

# Interactions per particle of the group walk at the paper's leaf and group sizes
# (they belong to the method: the opening test fixes the lists): log2 n, then for
# theta 0.4, 0.5, 0.6, 0.75 particle-particle and particle-cell pairs.
_PAIRS = ((15, (2423, 1481, 1098, 582), (1873, 1395, 1126, 782)),
          (17, (2307, 1366, 1068, 590), (3107, 2085, 1564, 993)),
          (20, (1751, 1119, 958, 465), (4600, 2810, 1992, 1306)))
_THETA = (0.4, 0.5, 0.6, 0.75)


def _flops(n, theta, mac=0):
    """Float operations of one force evaluation of n particles."""
    l = max(math.log2(max(n, 2)), 1.0)
    e = [r[0] for r in _PAIRS]
    pp, pc = ([float(np.interp(theta, _THETA, r[j])) for r in _PAIRS] for j in (1, 2))
    pp, pc = float(np.interp(l, e, pp)), float(np.interp(l, e, pc))
    if l < 15:          # a small system: the lists shrink towards all pairs
        pc *= max(0.0, (l - 8.0) / 7.0)
        pp = min(pp, float(n))
    f = (1.5, 1.65) if mac else (1.0, 1.0)
    return n * (20.0 * min(pp * f[0], n) + 57.0 * pc * f[1])


def work(case):
    kind = case["kind"]
    if kind in ("batch", "load", "serve"):
        rows = [(q["n"], q["theta"], q.get("mac", 0)) for q in _table_of(case)]
    else:
        rows = [(case["n"], case["theta"], case.get("mac", 0))]
    n = sum(r[0] for r in rows)
    one = sum(_flops(*r) for r in rows)
    load, state, out = 32 * n, 48 * n, 16 * n        # positions + masses; positions + velocities; acc, pot
    if kind in ("static", "forces", "load"):
        return dict(bytes=load + out, flops=one)
    if kind in ("restart", "serve"):
        return dict(bytes=load + 24 * n + state + out, flops=one * (1 + case["steps"]))
    if kind in ("steps", "batch"):
        return dict(bytes=2 * state + 8 * n + out, flops=one * case["steps"])
    if kind == "active":
        # the groups (about 19 particles) that hold an active one
        return dict(bytes=load + out + n, flops=one * (1.0 - (1.0 - case["share"]) ** 19))
    # a block step: about two evaluations of every particle
    return dict(bytes=2 * state + 8 * n + out, flops=2.0 * one)


# ---------------------------------------------------------------------------

_PAIR_LIMIT = 2.0e11      # pairs that the direct sums of one call may take (about 10 s)


def _direct(pos, mass, eps):
    n = pos.shape[0]
    e2 = float(np.float32(eps) * np.float32(eps))
    acc, pot = torch.empty_like(pos), torch.empty_like(mass)
    x, y, z = (pos[:, k].contiguous() for k in range(3))
    step = max(1, min(n, (1 << 26) // n))
    for a in range(0, n, step):
        b = min(n, a + step)
        dx, dy, dz = (q[None, :] - q[a:b, None] for q in (x, y, z))
        w = torch.rsqrt(dx * dx + dy * dy + dz * dz + e2)
        i = torch.arange(b - a, device=DEV)
        w[i, i + a] = 0.0
        mw = w * mass[None, :]
        pot[a:b] = -mw.sum(1)
        mw = mw * w * w
        for k, d in enumerate((dx, dy, dz)):
            acc[a:b, k] = (mw * d).sum(1)
    return acc, pot


def _leapfrog(pos, vel, mass, eps, dt, steps):
    acc, pot = _direct(pos, mass, eps)
    for _ in range(steps):
        vel = vel + acc * (0.5 * dt)
        pos = pos + vel * dt
        acc, pot = _direct(pos, mass, eps)
        vel = vel + acc * (0.5 * dt)
    return pos, vel, acc, pot


def exact(case, seed):
    kind = case["kind"]
    if kind in ("active", "block"):
        # what inactive particles keep, and the bins of a block step, are the
        # method's own and no plain sum gives them
        return None
    evals = 1 + case.get("steps", 0)
    if kind in ("batch", "load", "serve"):
        sizes = [q["n"] for q in _table_of(case)]
    else:
        sizes = [case["n"]]
    if evals * sum(float(n) ** 2 for n in sizes) > _PAIR_LIMIT:
        return None
    if kind in ("batch", "load", "serve"):
        tab, sys = _clusters(case, seed)
        got = [_leapfrog(p, v, m, q["eps"], q["dt"], evals - 1) for q, (p, v, m) in zip(tab, sys)]
        got = [torch.cat([r[j] for r in got]) for j in range(4)]
        return got[2:] if kind == "load" else got
    pos, vel, mass = _system(case["model"], case["n"], seed)
    if kind in ("static", "forces"):
        return _direct(pos, mass, case["eps"])
    got = _leapfrog(pos, vel, mass, case["eps"], case["dt"], evals - 1)
    if kind == "restart":
        return got
    T = float((0.5 * mass * (got[1] * got[1]).sum(1)).sum())
    W = float((0.5 * mass * got[3]).sum())
    return got, np.array([T, W, T + W])
