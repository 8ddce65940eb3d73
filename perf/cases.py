"""The work that a program has this library do, as measurable cases.

Every case is one call (or one forward and backward) through the package's
public functions on a synthetic Solar-System state: one force evaluation, a
run of velocity-Verlet steps, an ensemble of independent systems, the
differentiable trajectory with its gradients, and the conservation
diagnostics.  Sizes are those of the repository's own workloads (131, 2,079,
10,425 and 131,072 bodies, systems of 131 to 8,223 bodies in an ensemble) and
of its scans over N.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2112_15079_amd as nb
import solar_ics

DT = 0.1                       # days, the step of every workload
G = solar_ics.G_AU_DAY_MSUN


def listed():
    return [
        # one force evaluation of a small system: a program that has its own
        # integrator and calls the library once per stage (latency)
        {"name": "accel-131", "op": "accel", "n": 131, "precision": "fp64"},
        # the same call at the paper's body count, in the split form
        {"name": "accel-10425-split", "op": "accel", "n": 10425, "precision": "split"},
        # the planets, the Sun and a hundred asteroids for a tenth of a year
        {"name": "run-131", "op": "run", "n": 131, "steps": 365, "precision": "fp64"},
        # the low end of the N scan: a study of a thousand bodies
        {"name": "run-1000", "op": "run", "n": 1000, "steps": 100, "precision": "fp64"},
        # the accuracy study's 5,000 bodies
        {"name": "run-5000", "op": "run", "n": 5000, "steps": 100, "precision": "fp64"},
        # the paper's body count: the headline workload, between two outputs
        {"name": "run-10425", "op": "run", "n": 10425, "steps": 100, "precision": "fp64"},
        # the same in the split form
        {"name": "run-10425-split", "op": "run", "n": 10425, "steps": 100, "precision": "split"},
        # the largest system, a few steps between two outputs
        {"name": "run-131072", "op": "run", "n": 131072, "steps": 5, "precision": "fp64"},
        # an ensemble of systems of the ensemble workload's sizes
        {"name": "ensemble-24", "op": "ensemble", "systems": 24, "small": 131, "large": 8223,
         "steps": 10, "precision": "fp64"},
        # many small systems: variations of one planetary system
        {"name": "ensemble-128-small", "op": "ensemble", "systems": 128, "small": 40,
         "large": 400, "steps": 50, "precision": "fp64"},
        # a gradient step on initial conditions and masses (the adjoint
        # workload's system over two checkpoint intervals): forward and backward
        {"name": "grad-2079", "op": "grad", "n": 2079, "steps": 200, "every": 100},
        # the conservation check a run makes between its outputs
        {"name": "energy-10425", "op": "energy", "n": 10425},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Pair evaluations of the largest listed case: drawn runs stay below them.
_MOST_PAIRS = 6.0 * 131072.0 ** 2


def draw(rng):
    op = rng.choice(["accel", "run", "run", "run", "ensemble", "ensemble", "grad", "energy"])
    if op == "accel":
        return {"op": op, "n": _log_int(rng, 64, 131072),
                "precision": rng.choice(["fp64", "split"])}
    if op == "run":
        n = _log_int(rng, 64, 131072)
        most = max(1.0, min(365.0, 0.4 * _MOST_PAIRS / n ** 2))
        return {"op": op, "n": n, "steps": max(1, int(_log_int(rng, max(1.0, most / 20), most))),
                "precision": rng.choice(["fp64", "fp64", "split"])}
    if op == "ensemble":
        small = _log_int(rng, 33, 400)
        large = _log_int(rng, small + 1, 8223)
        return {"op": op, "systems": _log_int(rng, 3, 128 if large < 1500 else 24),
                "small": small, "large": large, "steps": _log_int(rng, 4, 50 if large < 1500 else 10),
                "precision": rng.choice(["fp64", "split"])}
    if op == "grad":
        n = _log_int(rng, 131, 10425)
        most = max(10.0, min(250.0, 0.05 * _MOST_PAIRS / n ** 2))
        return {"op": op, "n": n, "steps": _log_int(rng, most / 5, most),
                "every": rng.choice([10, 25, 50, 100])}
    return {"op": op, "n": _log_int(rng, 64, 131072)}


def _system(seed, n):
    """Sun, majors, and from 600 bodies up moons and heavy asteroids too."""
    if n >= 600:
        return solar_ics.solar_system(seed, n - 150, n_moons=100, n_heavy=19)
    return solar_ics.solar_system(seed, n - 31)


def _sizes(case):
    """The ensemble's system sizes: fixed by the case, not by the seed."""
    r = random.Random(case["systems"] * 100003 + case["small"] * 131 + case["large"])
    return [r.randint(case["small"], case["large"]) for _ in range(case["systems"])]


def _state(case, seed):
    """(pos, vel, mass) as numpy planes, and the ensemble's offsets."""
    if case["op"] == "ensemble":
        parts = [_system(seed * 1009 + k, n) for k, n in enumerate(_sizes(case))]
        cat = lambda f: np.concatenate([f(s) for s in parts], axis=-1)
        offs = [0]
        for s in parts:
            offs.append(offs[-1] + s.n)
        return cat(lambda s: s.pos), cat(lambda s: s.vel), cat(lambda s: s.mass), offs
    s = _system(seed, case["n"])
    return s.pos, s.vel, s.mass, None


def _cotangent(case, seed):
    """dL/dr_T and dL/dv_T of a program's loss, known before the call."""
    r = np.random.default_rng(seed + 7)
    return r.normal(0.0, 1.0, (3, case["n"])), r.normal(0.0, 1.0, (3, case["n"]))


def prepare(case, seed):
    pos, vel, mass, offs = _state(case, seed)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    st = {"case": case, "pos": dev(pos), "vel": dev(vel), "mass": dev(mass), "offsets": offs}
    if case["op"] == "grad":
        st["gr"], st["gv"] = (dev(a) for a in _cotangent(case, seed))
        for k in ("pos", "vel", "mass"):
            st[k].requires_grad_()
    return st


def run(st):
    c = st["case"]
    if c["op"] == "accel":
        return nb.accel(st["pos"], st["mass"], G, precision=c["precision"])
    if c["op"] == "run":
        return nb.verlet_run(st["pos"], st["vel"], st["mass"], G, DT, c["steps"],
                             precision=c["precision"])
    if c["op"] == "ensemble":
        return nb.verlet_run_batched(st["pos"], st["vel"], st["mass"], st["offsets"], G, DT,
                                     c["steps"], precision=c["precision"])
    if c["op"] == "grad":
        r, v = nb.verlet(st["pos"], st["vel"], st["mass"], G, DT, c["steps"],
                         checkpoint_every=c["every"])
        grads = torch.autograd.grad((r, v), (st["pos"], st["vel"], st["mass"]),
                                    (st["gr"], st["gv"]))
        return [r.detach(), v.detach(), *grads]
    return [nb.energy(st["pos"], st["vel"], st["mass"], G),
            nb.momenta(st["pos"], st["vel"], st["mass"])]


def work(case):
    """Each unordered pair once: 20 operations for the pair's term and 7 for
    the reaction; a gradient step runs each step forward, and back once more
    with its transposed Jacobian (47 per pair and 19 for the other body)."""
    ns = _sizes(case) if case["op"] == "ensemble" else [case["n"]]
    bodies, pairs = sum(ns), sum(n * (n - 1) / 2.0 for n in ns)
    if case["op"] == "accel":
        return {"bytes": 8.0 * 7 * bodies, "flops": 27.0 * pairs}
    if case["op"] in ("run", "ensemble"):
        return {"bytes": 8.0 * 13 * bodies, "flops": 27.0 * pairs * (case["steps"] + 1)}
    if case["op"] == "grad":
        return {"bytes": 8.0 * 26 * bodies, "flops": (27.0 + 66.0) * pairs * (case["steps"] + 1)}
    return {"bytes": 8.0 * 7 * bodies, "flops": 12.0 * pairs}


# ----------------------------------------------------------------------------
# the same in plain torch, 64 bits

def _accel64(pos, mass):
    """Eq. (1) by rows of targets, a block of rows at a time."""
    n = mass.shape[0]
    rows = max(1, min(n, (1 << 26) // n))
    out = []
    for p0 in range(0, n, rows):
        p1 = min(p0 + rows, n)
        d = [pos[k][None, :] - pos[k][p0:p1, None] for k in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        own = torch.arange(p0, p1, device=pos.device)
        eye = torch.zeros_like(r2)
        eye[own - p0, own] = 1.0
        f = (G * mass)[None, :] * (1.0 - eye) / ((r2 + eye) * torch.sqrt(r2 + eye))
        out.append(torch.stack([(f * x).sum(1) for x in d]))
    return torch.cat(out, dim=1)


def _step64(pos, vel, acc, mass):
    """Eqs. (3)-(4)."""
    r = pos + DT * vel + (0.5 * DT * DT) * acc
    a = _accel64(r, mass)
    return r, vel + (0.5 * DT) * (acc + a), a


def _run64(pos, vel, mass, steps):
    acc = _accel64(pos, mass)
    for _ in range(steps):
        pos, vel, acc = _step64(pos, vel, acc, mass)
    return pos, vel


def _grad64(pos, vel, mass, gr, gv, steps):
    """Reverse sweep over the stored states, one step's graph at a time."""
    states = [(pos, vel, _accel64(pos, mass))]
    for _ in range(steps):
        states.append(_step64(*states[-1], mass))
    lr, lv, la, gm = gr, gv, torch.zeros_like(gr), torch.zeros_like(mass)
    for s in reversed(states[:-1]):
        x = [t.detach().requires_grad_() for t in (*s, mass)]
        lr, lv, la, dm = torch.autograd.grad(_step64(*x), x, (lr, lv, la))
        gm = gm + dm
    x = [pos.detach().requires_grad_(), mass.detach().requires_grad_()]
    dr, dm = torch.autograd.grad(_accel64(*x), x, la)
    return [states[-1][0], states[-1][1], lr + dr, lv, gm + dm]


def _energy64(pos, vel, mass):
    n, pot = mass.shape[0], torch.zeros((), dtype=torch.float64, device=pos.device)
    rows = max(1, min(n, (1 << 26) // n))
    for p0 in range(0, n, rows):
        p1 = min(p0 + rows, n)
        d = [pos[k][None, :] - pos[k][p0:p1, None] for k in range(3)]
        r = torch.sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2])
        own = torch.arange(p0, p1, device=pos.device)
        r[own - p0, own] = math.inf
        pot = pot - 0.5 * G * (mass[p0:p1] * (mass[None, :] / r).sum(1)).sum()
    kin = 0.5 * (mass * (vel * vel).sum(0)).sum()
    p = (mass * vel).sum(1)
    l = (mass * torch.linalg.cross(pos, vel, dim=0)).sum(1)
    return [torch.stack([kin, pot, kin + pot]), torch.cat([p, l])]


def exact(case, seed):
    pos, vel, mass, offs = _state(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    pos, vel, mass = t(pos), t(vel), t(mass)
    if case["op"] == "accel":
        return _accel64(pos, mass)
    if case["op"] == "run":
        return _run64(pos, vel, mass, case["steps"])
    if case["op"] == "ensemble":
        r, v = torch.empty_like(pos), torch.empty_like(vel)
        for a, b in zip(offs, offs[1:]):
            r[:, a:b], v[:, a:b] = _run64(pos[:, a:b], vel[:, a:b], mass[a:b], case["steps"])
        return r, v
    if case["op"] == "grad":
        gr, gv = (t(a) for a in _cotangent(case, seed))
        return _grad64(pos, vel, mass, gr, gv, case["steps"])
    return _energy64(pos, vel, mass)
