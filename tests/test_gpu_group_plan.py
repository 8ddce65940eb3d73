"""The work list of an ensemble in the workgroups that stay on the chip: a first
call on new offsets, which builds it, takes no longer than one by launches
(chosen by setting the tile), whose list is simpler."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")
from paper_2112_15079_amd import _capi as C  # noqa: E402

DEV = "cuda:0"


def call(offs, state, steps=1):
    """The call itself, from offsets in host memory; returns its time."""
    n, ns = int(offs[-1]), len(offs) - 1
    need = C.workspace_bytes(C.OP_BATCHED, n, num_systems=ns, steps=steps)
    ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    t = time.perf_counter()
    st = C.load().nbody_verlet_run_batched(*[x.data_ptr() for x in state], offs.ctypes.data, ns,
                                           1e-4, 0.1, steps, C.NBODY_FP64, 0.0, ws.data_ptr(),
                                           ws.numel(), C.stream_handle(DEV))
    torch.cuda.synchronize()
    assert st == C.NBODY_OK, C.last_error()
    return time.perf_counter() - t


@pytest.mark.parametrize("ns", [2000, 20000, 200000])
def test_first_call_on_new_offsets(ns):
    r = np.random.default_rng(ns)
    times = {}
    for route in ("here", "by launches"):
        nb.reset_caches()
        if route == "by launches":
            nb.set_tile(2, "fp64", 0, *nb.get_tile(2, "fp64", 0).values())
        times[route] = 1e9
        for _ in range(5):   # (the first of them loads the kernels)
            offs = np.concatenate([[0], np.cumsum(r.integers(3, 40, ns))]).astype(np.int64)
            n = int(offs[-1])
            state = [torch.rand(3, n, dtype=torch.float64, device=DEV),
                     torch.zeros(3, n, dtype=torch.float64, device=DEV),
                     torch.full((n,), 1e-9, dtype=torch.float64, device=DEV)]
            times[route] = min(times[route], call(offs, state))
    nb.reset_caches()
    assert times["here"] <= 1.2 * times["by launches"], times


@pytest.mark.parametrize("ns,m", [(280, 998), (300, 899), (282, 862)])
def test_large_uniform_ensembles(ns, m):
    """Sizes whose shares fill the chip badly: no slower than by launches."""
    offs = np.arange(ns + 1, dtype=np.int64) * m
    state = [torch.rand(3, ns * m, dtype=torch.float64, device=DEV),
             torch.zeros(3, ns * m, dtype=torch.float64, device=DEV),
             torch.full((ns * m,), 1e-12, dtype=torch.float64, device=DEV)]
    times = [1e9, 1e9]
    for _ in range(4):   # (in turn, so that the clock's rise favours neither)
        for route in (0, 1):
            nb.reset_caches()
            if route:
                nb.set_tile(2, "fp64", 0, *nb.get_tile(2, "fp64", 0).values())
            call(offs, state, 20)
            times[route] = min(times[route], *(call(offs, state, 20) for _ in range(3)))
    nb.reset_caches()
    assert times[0] <= 1.15 * times[1], times   # (here, by launches)


@pytest.mark.parametrize("ns", [1 << 22, (1 << 22) + 1, 17_000_000])
def test_more_systems_than_a_launch_has_threads_for(ns):
    """Single bodies drift: a launch of 2^32 threads holds 16.7 million workgroups of
    256, so many systems go by launches."""
    nb.reset_caches()
    offs = np.arange(ns + 1, dtype=np.int64)
    pos = torch.rand(3, ns, dtype=torch.float64, device=DEV)
    vel = torch.rand(3, ns, dtype=torch.float64, device=DEV)
    mass = torch.full((ns,), 1e-9, dtype=torch.float64, device=DEV)
    # (the drift is a fused multiply-add: half an ulp of the result from this)
    want = pos + 0.1 * vel + 0.1 * vel
    call(offs, [pos, vel, mass], steps=2)
    assert bool((torch.abs(pos - want) <= 2 ** -51 * want).all())
    nb.reset_caches()
