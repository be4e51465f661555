"""Timed cases of the library: the calls a user's program makes, from the
smallest to the largest sizes, in every precision.

Inputs are Plummer spheres in Henon units made on the GPU from a seed (the
shape of every workload of ``bench.py``).  ``run`` is one pass through the
public entry points of ``Context`` and ``BlockIntegrator``.
"""
import math

import numpy as np
import torch

import paper_1409_5474_amd as nb
from paper_1409_5474_amd.integrator import BlockIntegrator

PRECISIONS = ("fp64", "mixed", "mixed_ds")
ETA = 0.01
# force evaluations per particle and time unit of a Plummer sphere integrated
# with eta = 0.01 and eps = 1/256 (65536 bodies to t = 1/8: 2.47e11 pairs)
EVALS_PER_TIME = 460.0


def listed():
    return [
        # an interactive or test-sized cluster, every particle active: latency and launches count
        dict(name="forces_fp64_1024", kind="forces", prec="fp64", n=1024, active=1024),
        # the benchmark's headline: all-active mixed evaluation
        dict(name="forces_mixed_262144", kind="forces", prec="mixed", n=262144, active=262144),
        # a mid-size system of odd length, start-up or energy evaluation in double precision
        dict(name="forces_fp64_40009", kind="forces", prec="fp64", n=40009, active=40009),
        # one block of a block-step integration driven by the caller: few active rows of many particles
        dict(name="forces_ds_65537_few", kind="forces", prec="mixed_ds", n=65537, active=1117),
        # coupling kick of the Hamiltonian split: a cluster's members in the field of a galaxy
        dict(name="cross_mixed_1000003", kind="cross", prec="mixed", n=1000003, active=3899),
        # all-active evaluation of many independent clusters
        dict(name="batch_mixed_128", kind="batch", prec="mixed", systems=128, n_min=128, n_max=16384),
        # the sixth-order scheme's forces with snap
        dict(name="forces6_20011", kind="forces6", prec="fp64", n=20011, active=20011),
        # collisionless field, start of a run of a small and of a large galaxy
        dict(name="tree_fp64_10007", kind="tree", prec="fp64", n=10007, theta=0.5),
        dict(name="tree_mixed_262144", kind="tree", prec="mixed", n=262144, theta=0.5),
        # whole block-step runs to a synchronisation time: the split's small cluster, a large cluster, a batch
        dict(name="steps_fp64_3899", kind="steps", prec="fp64", n=3899, dt_max=1.0 / 16),
        dict(name="steps_fp64_65536", kind="steps", prec="fp64", n=65536, dt_max=1.0 / 64),
        dict(name="steps_batch_mixed_24", kind="steps_batch", prec="mixed", systems=24, n_min=128, n_max=8192,
             dt_max=1.0 / 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "forces", "cross", "batch", "forces6", "tree", "tree", "steps", "steps",
                       "steps_batch"])
    if kind == "forces":
        prec = rng.choice(PRECISIONS)
        n = _log_int(rng, 700, 160000 if prec == "fp64" else 250000)
        return dict(kind=kind, prec=prec, n=n, active=n if rng.random() < 0.5 else _log_int(rng, 3, n))
    if kind == "cross":
        n = _log_int(rng, 20000, 1000000)
        return dict(kind=kind, prec=rng.choice(("fp64", "mixed")), n=n, active=_log_int(rng, 100, 4000))
    if kind == "batch":
        return dict(kind=kind, prec=rng.choice(PRECISIONS), systems=_log_int(rng, 8, 128), n_min=128,
                    n_max=_log_int(rng, 1024, 16384))
    if kind == "forces6":
        n = _log_int(rng, 700, 40000)
        return dict(kind=kind, prec="fp64", n=n, active=n if rng.random() < 0.6 else _log_int(rng, 20, n))
    if kind == "tree":
        return dict(kind=kind, prec=rng.choice(("fp64", "mixed")), n=_log_int(rng, 2000, 250000),
                    theta=rng.choice((0.4, 0.5, 0.6, 0.75)))
    if kind == "steps":
        n = _log_int(rng, 1024, 60000)
        return dict(kind=kind, prec=rng.choice(("fp64", "fp64", "mixed")), n=n,
                    dt_max=1.0 / 16 if n <= 16384 else 1.0 / 64)
    return dict(kind="steps_batch", prec=rng.choice(("fp64", "mixed")), systems=_log_int(rng, 4, 32), n_min=128,
                n_max=_log_int(rng, 512, 8192), dt_max=1.0 / 64)


# ---------------------------------------------------------------- inputs ----
def _plummer(n, gen):
    """A Plummer sphere of n equal masses summing to 1 (cut at ten scale
    radii, isotropic Gaussian velocities of the local dispersion), centre of
    mass at rest."""
    f = dict(dtype=torch.float64, device="cuda", generator=gen)

    def directions():
        z = 2.0 * torch.rand(n, **f) - 1.0
        phi = 2.0 * math.pi * torch.rand(n, **f)
        rho = torch.sqrt(1.0 - z * z)
        return torch.stack([rho * torch.cos(phi), rho * torch.sin(phi), z], 1)

    m_cut = (10.0 / math.sqrt(101.0)) ** 3
    x = (1e-9 + (1.0 - 1e-9) * torch.rand(n, **f)) * m_cut
    r = 1.0 / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    sigma = torch.sqrt(1.0 / (6.0 * torch.sqrt(1.0 + r * r)))
    pos = (3.0 * math.pi / 16.0) * r[:, None] * directions()
    vel = math.sqrt(16.0 / (3.0 * math.pi)) * sigma[:, None] * torch.randn((n, 3), **f)
    pos -= pos.mean(0)
    vel -= vel.mean(0)
    return pos.contiguous(), vel.contiguous(), torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")


def _active(n, k, gen):
    if k >= n:
        return torch.arange(n, dtype=torch.int32, device="cuda")
    return torch.randperm(n, device="cuda", generator=gen)[:k].sort().values.to(torch.int32)


def _sizes(case):
    """Log-spaced system sizes of a batch, the same for every seed."""
    c = case["systems"]
    u = (np.arange(c) * 0.6180339887498949 + 0.5) % 1.0
    s = np.floor(case["n_min"] * (case["n_max"] / case["n_min"]) ** u).astype(np.int64)
    return np.concatenate([[0], np.cumsum(s)])


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    d = {}
    if kind in ("batch", "steps_batch"):
        off = _sizes(case)
        parts = [_plummer(int(off[c + 1] - off[c]), gen) for c in range(len(off) - 1)]
        d["pos"], d["vel"], d["mass"] = (torch.cat([p[k] for p in parts]) for k in range(3))
        d["offsets"] = off
        d["eps2"] = (0.05 * np.diff(off).astype(np.float64) ** (-1.0 / 3.0)) ** 2
        return d
    d["pos"], d["vel"], d["mass"] = _plummer(case["n"], gen)
    d["eps2"] = 1.0 / 256 ** 2
    if kind == "cross":
        d["pos_i"], d["vel_i"], _ = _plummer(case["active"], gen)
        d["pos_i"] *= 0.25
        d["active"] = torch.arange(case["active"], dtype=torch.int32, device="cuda")
    elif "active" in case:
        d["active"] = _active(case["n"], case["active"], gen)
    if kind == "forces6":
        # accelerations of the size the sphere's own field has
        r2 = (d["pos"] ** 2).sum(1, keepdim=True)
        d["acc_j"] = -d["pos"] * (r2 + 0.35) ** -1.5
    return d


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    s["ctx"] = nb.Context(0, case["prec"])
    if kind in ("steps", "steps_batch"):
        bi = BlockIntegrator(s["ctx"], s["pos"], s["vel"], s["mass"], s["eps2"], eta=ETA, dt_max=case["dt_max"],
                             offsets=s.get("offsets"))
        s["run"] = bi
        s["start"] = {k: getattr(bi, k).clone() for k in ("pos", "vel", "acc", "jerk", "t_tick", "level", "sched")}
    elif kind == "batch":
        n = int(s["offsets"][-1])
        s["active"] = torch.arange(n, dtype=torch.int32, device="cuda")
        s["out"] = (torch.empty((n, 3), dtype=torch.float64, device="cuda"),
                    torch.empty((n, 3), dtype=torch.float64, device="cuda"),
                    torch.empty(n, dtype=torch.float64, device="cuda"))
    return s


# ------------------------------------------------------------------- run ----
def run(state):
    s, ctx, kind = state, state["ctx"], state["case"]["kind"]
    if kind == "forces":
        return ctx.forces(s["pos"], s["vel"], s["mass"], s["active"], s["eps2"])
    if kind == "cross":
        return ctx.forces_ij(s["pos"], s["vel"], s["mass"], s["pos_i"], s["vel_i"], s["active"], s["eps2"])
    if kind == "forces6":
        return ctx.forces6(s["pos"], s["vel"], s["acc_j"], s["mass"], s["active"], s["eps2"])
    if kind == "batch":
        return ctx.forces_batch(s["offsets"], s["eps2"], s["pos"], s["vel"], s["mass"], s["active"], s["offsets"],
                                *s["out"])
    if kind == "tree":
        acc, pot, _ = ctx.tree_forces(s["pos"], s["mass"], s["eps2"], theta=s["case"]["theta"], stats=False)
        return acc, pot
    # a run from its start state to the first synchronisation time
    bi = s["run"]
    for k, v in s["start"].items():
        getattr(bi, k).copy_(v)
    bi.run_until(s["case"]["dt_max"])
    return bi.pos, bi.vel, bi.acc, bi.jerk, bi.t_tick, bi.level


def work(case):
    kind = case["kind"]
    if kind in ("batch", "steps_batch"):
        sizes = np.diff(_sizes(case)).astype(np.float64)
        n, pairs = float(sizes.sum()), float((sizes ** 2).sum())
        if kind == "batch":
            return dict(bytes=(56 + 4 + 56) * n, flops=43.0 * pairs)
        evals = EVALS_PER_TIME * case["dt_max"]
        return dict(bytes=2 * (4 * 24 + 12) * n, flops=43.0 * pairs * evals)
    n = float(case["n"])
    if kind == "steps":
        return dict(bytes=2 * (4 * 24 + 12) * n, flops=43.0 * n * n * EVALS_PER_TIME * case["dt_max"])
    if kind == "tree":
        # cells and leaf particles met per particle
        cells = 180.0 * math.log2(n) * (0.5 / case["theta"]) ** 2
        return dict(bytes=(32 + 32) * n, flops=n * (40.0 * cells + 20.0 * 1.3 * cells))
    a = float(case["active"])
    if kind == "forces6":
        return dict(bytes=80 * n + 4 * a + 80 * a, flops=80.0 * n * a)
    return dict(bytes=56 * n + 4 * a + 56 * a + (48 * a if kind == "cross" else 0), flops=43.0 * n * a)


# ----------------------------------------------------------------- exact ----
def _direct(pos, vel, mass, xi, vi, rows, eps2, acc_j=None, ai=None):
    """Acceleration, jerk (with vel), snap (with acc_j) and potential of the
    receivers xi by plain 64-bit sums; ``rows``: their own rows among the
    sources (None: none of them is a source)."""
    ni, n = xi.shape[0], pos.shape[0]
    acc = torch.empty_like(xi)
    jerk = torch.empty_like(xi) if vel is not None else None
    snap = torch.empty_like(xi) if acc_j is not None else None
    pot = torch.empty(ni, dtype=torch.float64, device=xi.device)
    step = max(1, (1 << 26) // n)
    for b in range(0, ni, step):
        e = min(ni, b + step)
        r = [pos[:, c][None, :] - xi[b:e, c][:, None] for c in range(3)]
        s = r[0] * r[0]
        s.addcmul_(r[1], r[1]).addcmul_(r[2], r[2]).add_(eps2)
        q2 = 1.0 / s
        mq = torch.sqrt(q2).mul_(mass[None, :])
        if rows is not None:
            mq[torch.arange(e - b, device=xi.device), rows[b:e].long()] = 0.0
        pot[b:e] = -mq.sum(1)
        mq3 = mq.mul_(q2)
        for c in range(3):
            acc[b:e, c] = (mq3 * r[c]).sum(1)
        if vel is None:
            continue
        u = [vel[:, c][None, :] - vi[b:e, c][:, None] for c in range(3)]
        alpha = (r[0] * u[0]).addcmul_(r[1], u[1]).addcmul_(r[2], u[2]).mul_(q2)
        if acc_j is not None:
            beta = (u[0] * u[0]).addcmul_(u[1], u[1]).addcmul_(u[2], u[2])
            w = [acc_j[:, c][None, :] - ai[b:e, c][:, None] for c in range(3)]
            for c in range(3):
                beta.addcmul_(r[c], w[c])
            beta.mul_(q2).addcmul_(alpha, alpha)
        for c in range(3):
            uc = torch.addcmul(u[c], alpha, r[c], value=-3.0)
            jerk[b:e, c] = (mq3 * uc).sum(1)
            if acc_j is not None:
                wc = w[c].addcmul_(alpha, uc, value=-6.0).addcmul_(beta, r[c], value=-3.0)
                snap[b:e, c] = (mq3 * wc).sum(1)
    return acc, jerk, snap, pot


def _hermite(pos, vel, mass, eps2, dt_max, max_level=30):
    """Block-step Hermite integration of one system to t = dt_max."""
    n = pos.shape[0]
    x, v = pos.clone(), vel.clone()
    every = torch.arange(n, device=x.device)
    a, j, _, _ = _direct(x, v, mass, x, v, every, eps2)
    norm = lambda y: torch.sqrt((y * y).sum(1))
    lev = torch.ceil(-torch.log2(ETA * norm(a) / norm(j) / dt_max)).clamp_(0, max_level).long()
    full = 1 << max_level
    tick = dt_max / full
    t = torch.zeros(n, dtype=torch.int64, device=x.device)
    while True:
        end = t + (full >> lev)
        nxt = end.min()
        if int(nxt) > full:
            return x, v, a, j
        act = (end == nxt).nonzero()[:, 0]
        d = ((nxt - t).double() * tick)[:, None]
        xp = x + d * (v + d * (0.5 * a + d * (j / 6.0)))
        vp = v + d * (a + d * (0.5 * j))
        a1, j1, _, _ = _direct(xp, vp, mass, xp[act], vp[act], act, eps2)
        h = (dt_max / 2.0 ** lev[act].double())[:, None]
        a0, j0 = a[act], j[act]
        a2 = (-6.0 * (a0 - a1) - h * (4.0 * j0 + 2.0 * j1)) / h ** 2
        a3 = (12.0 * (a0 - a1) + 6.0 * h * (j0 + j1)) / h ** 3
        x[act] = xp[act] + a2 * h ** 4 / 24.0 + a3 * h ** 5 / 120.0
        v[act] = vp[act] + a2 * h ** 3 / 6.0 + a3 * h ** 4 / 24.0
        a[act], j[act], t[act] = a1, j1, nxt
        a2e = a2 + a3 * h
        want = torch.sqrt(ETA * (norm(a1) * norm(a2e) + norm(j1) ** 2) / (norm(j1) * norm(a3) + norm(a2e) ** 2))
        h, l0 = h[:, 0], lev[act]
        down = torch.ceil(torch.log2(h / want)).clamp_(min=0).long()
        up = (want >= 2.0 * h) & (l0 > 0) & (nxt % (2 * (full >> l0)) == 0)
        lev[act] = torch.where(h > want, (l0 + down).clamp_(max=max_level), l0 - up.long())
        # every particle has reached the end: the next step lies beyond it
        if int(t.min()) >= full:
            return x, v, a, j


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "steps":
        return (*_hermite(d["pos"], d["vel"], d["mass"], d["eps2"], case["dt_max"]), None, None)
    if kind in ("batch", "steps_batch"):
        off, out = d["offsets"], []
        for c in range(len(off) - 1):
            p, v, m = (d[k][off[c]:off[c + 1]] for k in ("pos", "vel", "mass"))
            if kind == "batch":
                a, j, _, w = _direct(p, v, m, p, v, torch.arange(len(m), device=p.device), float(d["eps2"][c]))
                out.append((a, j, w))
            else:
                out.append(_hermite(p, v, m, float(d["eps2"][c]), case["dt_max"]))
        got = tuple(torch.cat(x) for x in zip(*out))
        return got if kind == "batch" else (*got, None, None)
    if kind == "cross":
        a, j, _, w = _direct(d["pos"], d["vel"], d["mass"], d["pos_i"], d["vel_i"], None, d["eps2"])
        return a, j, w
    if kind == "tree":
        # the sums that the multipole expansion approximates
        n = case["n"]
        a, _, _, w = _direct(d["pos"], None, d["mass"], d["pos"], None, torch.arange(n, device="cuda"), d["eps2"])
        return a, w
    act = d["active"].long()
    a, j, s, w = _direct(d["pos"], d["vel"], d["mass"], d["pos"][act], d["vel"][act], act, d["eps2"],
                         d.get("acc_j"), d["acc_j"][act] if kind == "forces6" else None)
    return (a, j, s, w) if kind == "forces6" else (a, j, w)
