"""Runs and reverse sweeps that stay on the chip when workgroups come late (test
instrument tests/host/libgroupprobe.so, the library's own kernels): one
workgroup that does everything, a few that are joined while the run goes on,
half of them.  Each gives the result of a full launch bit for bit, and that is the
library's.  And runs at once, which the library starts as they come, take about
as long as one after the other."""
import ctypes
import os
import time

import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "tests", "host", "libgroupprobe.so")
DEV = "cuda:0"
STEPS = 21
NEVER = 1 << 20


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.fixture(scope="module")
def lib():
    assert os.path.exists(LIB), f"{LIB} is missing: run __graft_entry__.build()"
    lib = ctypes.CDLL(LIB)
    P, I, L, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_double
    lib.group_probe_run.argtypes = [I, I, I, I, I, I, P, P, P, L, P, D, D, L, P, P, P, P, P]
    lib.group_probe_sweep.argtypes = [I, I, I, I, I, I, I, P, P, P, P, P, P, L, D, D, L, P, P, P]
    return lib


def scratch(n):
    return (torch.zeros(12 * n, dtype=torch.float64, device=DEV),
            torch.zeros(4, dtype=torch.int32, device=DEV))


def lateness(groups):
    """(workgroups on time, launch indices between arrivals)"""
    return [(groups, 0), (1, NEVER), (min(3, groups - 1), 2), (groups // 2, 3), (1, 1),
            (groups - 1, 3)]


def check_joined(reg, groups, on_time, step):
    torch.cuda.synchronize()
    count, began, _, word_hi = reg.cpu().numpy()
    assert began <= on_time
    if step == NEVER:
        assert began == on_time and word_hi == -1       # the run ended without them
    elif on_time < groups:
        assert count == groups and 0 < word_hi < STEPS   # all of them joined


def run(lib, s, n, shape, nmaj, on_time, step, traj=None):
    spread = 8 if n <= 256 else 1
    groups = -(-n // (shape[0] * shape[1]))
    p, v, m = T(s.pos), T(s.vel), T(s.mass)
    xbuf, reg = scratch(n)
    flags = torch.zeros(1, dtype=torch.int32, device=DEV)
    rc = lib.group_probe_run(*shape, spread, on_time * spread, step, p.data_ptr(), v.data_ptr(),
                             m.data_ptr(), n, nmaj.data_ptr() if nmaj is not None else None, s.G,
                             0.1, STEPS, traj.data_ptr() if traj is not None else None,
                             xbuf.data_ptr(), reg.data_ptr(), flags.data_ptr(), None)
    assert rc == 0
    check_joined(reg, groups, on_time, step)
    assert flags.item() == 0
    return p, v


RUNS = [(131, (1, 8, 512)), (700, (1, 4, 512)), (1000, (1, 4, 1024)), (1100, (1, 5, 1024)),
        (1400, (2, 3, 512)), (2000, (2, 4, 512)), (2079, (3, 3, 512)), (2500, (2, 5, 1024)),
        (3000, (3, 4, 1024)), (4095, (4, 4, 512))]


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("n,shape", RUNS)
def test_run_with_late_workgroups(lib, n, shape, split):
    s = S.solar_system(n % 7, n - 31)
    nmaj = torch.tensor([n // 9], dtype=torch.int64, device=DEV) if split else None
    groups = -(-n // (shape[0] * shape[1]))
    if not split:   # (the library has its own order of the bodies in the split form)
        nb.reset_caches()
        want = T(s.pos), T(s.vel)
        nb.verlet_run(*want, T(s.mass), s.G, 0.1, STEPS)
    else:
        want = run(lib, s, n, shape, nmaj, groups, 0)
    for on_time, step in lateness(groups):
        p, v = run(lib, s, n, shape, nmaj, on_time, step)
        assert torch.equal(p, want[0]) and torch.equal(v, want[1]), (on_time, step)


@pytest.mark.parametrize("n,shape,held", [
    (131, (1, 8, 512), 1), (700, (1, 4, 512), 1), (1250, (1, 5, 512), 1), (1500, (2, 3, 512), 1),
    (1600, (2, 4, 512), 1), (2000, (2, 4, 512), 0), (2079, (2, 5, 512), 0), (2500, (5, 2, 512), 0),
    (3000, (3, 4, 512), 0), (4095, (4, 4, 512), 0)])
def test_sweep_with_late_workgroups(lib, n, shape, held):
    s = S.solar_system(n % 7, n - 31)
    traj = torch.zeros((STEPS + 1, 3, n), dtype=torch.float64, device=DEV)
    run(lib, s, n, dict(RUNS).get(n, (4, 4, 512)), None, 10 ** 6, 0, traj)
    seg = torch.cat([T(s.pos)[None], traj[:STEPS]]).contiguous()   # r_0 .. r_STEPS
    r = np.random.default_rng(n)
    lr, lv = r.standard_normal((3, n)), r.standard_normal((3, n))
    mass = T(s.mass)
    spread = 8 if n <= 256 else 1
    groups = -(-n // (shape[0] * shape[1]))
    want = None
    for on_time, step in lateness(groups):
        g = [T(lr), T(lv), torch.zeros(n, dtype=torch.float64, device=DEV)]
        xbuf, reg = scratch(n)
        rc = lib.group_probe_sweep(*shape, held, spread, on_time * spread, step, seg.data_ptr(),
                                   seg[STEPS].data_ptr(), mass.data_ptr(), *[x.data_ptr() for x in g],
                                   n, s.G, 0.1, STEPS + 1, xbuf.data_ptr(), reg.data_ptr(), None)
        assert rc == 0
        check_joined(reg, groups, on_time, step)
        assert all(torch.isfinite(x).all() for x in g)
        want = want or g
        assert all(torch.equal(a, b) for a, b in zip(g, want)), (on_time, step)


@pytest.mark.parametrize("n,steps,runs,times", [(1000, 1000, 2, 6), (4000, 500, 2, 6),
                                                (1000, 400, 4, 8)])
def test_runs_at_once_do_not_starve_each_other(n, steps, runs, times):
    """The later of several runs begin on what the first leaves of the chip.  They must
    have the chip when the first has ended: all take about as long as one after
    the other.  (When the workgroups that came late left for good, two took 24 and
    32 times as long as one.)"""
    nb.reset_caches()
    states = [S.solar_system(k, n - 31) for k in range(runs)]
    args = [(T(s.pos), T(s.vel), T(s.mass)) for s in states]
    streams = [torch.cuda.Stream() for _ in range(runs)]

    def timed(k):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for a, st in list(zip(args, streams))[:k]:
            with torch.cuda.stream(st):
                nb.verlet_run(*a, S.G_AU_DAY_MSUN, 0.1, steps)
        torch.cuda.synchronize()
        return time.perf_counter() - t

    for k in (1, runs):
        timed(k)   # (kernels loaded, workspaces made)
    one = min(timed(1) for _ in range(3))
    together = min(timed(runs) for _ in range(3))
    assert together <= times * one, (one, together)
