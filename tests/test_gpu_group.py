"""Runs by workgroups that stay on the chip and exchange positions (single
systems of 80 to 4,095 bodies): at the sizes where the launch shape changes,
against the oracle; chaining; more steps than one launch holds; under graph
capture; and beside work that holds the GPU, when part of the workgroups
comes late."""
import numpy as np
import pytest
import torch

import oracle
import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")
from paper_2112_15079_amd import _capi as C  # noqa: E402

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def H(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def rel(a, b):
    return float(np.max(np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)))


def run(s, parts, precision="fp64"):
    p, v, m = T(s.pos), T(s.vel), T(s.mass)
    for k in parts:
        nb.verlet_run(p, v, m, s.G, s.dt, k, precision=precision)
    return H(p), H(v)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("split", 2e-12)])
@pytest.mark.parametrize("n", [79, 80, 83, 256, 257, 768, 769, 1021, 1024, 1025, 2048, 2049,
                               3072, 3073, 4095])
def test_shapes_match_oracle_and_chain(n, precision, tol):
    nb.reset_caches()
    s = S.solar_system(70 + n % 7, n - 31)
    a = H(nb.accel(T(s.pos), T(s.mass), s.G, precision=precision))
    assert rel(a, oracle.accel(s.pos, s.mass, s.G)) <= tol
    p, v = run(s, [12], precision)
    p2, v2 = run(s, [5, 1, 6], precision)
    assert np.array_equal(p, p2) and np.array_equal(v, v2)
    pr, vr = oracle.verlet(s.pos, s.vel, s.mass, s.G, s.dt, 12)
    assert rel(p[:, 1:], pr[:, 1:]) <= 1e-10 and rel(v[:, 1:], vr[:, 1:]) <= 1e-10


def test_more_steps_than_one_launch():
    """2,100 steps are three launches; the same run in pieces is equal bit for
    bit, and within the year-long run's bar of the oracle."""
    s = S.solar_system(71, 100 - 31)
    p, v = run(s, [2100])
    p2, v2 = run(s, [1023, 1, 1076])
    assert np.array_equal(p, p2) and np.array_equal(v, v2)
    pr, _ = oracle.verlet(s.pos, s.vel, s.mass, s.G, s.dt, 2100)
    assert rel(p[:, 1:], pr[:, 1:]) <= 1e-10


@pytest.mark.parametrize("n", [150, 1500])
def test_split_classes_that_straddle_a_workgroup(n):
    """Heavy bodies: none, one, a count inside a workgroup's targets, all."""
    s = S.solar_system(72, n - 31)
    ref = oracle.accel(s.pos, s.mass, s.G)
    order = np.sort(s.mass)[::-1]
    for k in (0, 1, 5, 13, n):
        thr = 10.0 if k == 0 else float(order[k - 1])
        a = H(nb.accel(T(s.pos), T(s.mass), s.G, precision="split", small_mass=thr))
        # with the Sun among the light sources every term is FP32
        assert rel(a, ref) <= (2e-6 if k == 0 else 2e-7)
        p, v, m = T(s.pos), T(s.vel), T(s.mass)
        nb.verlet_run(p, v, m, s.G, s.dt, 6, precision="split", small_mass=thr)
        q, w = T(s.pos), T(s.vel)
        for _ in range(2):
            nb.verlet_run(q, w, m, s.G, s.dt, 3, precision="split", small_mass=thr)
        assert np.array_equal(H(p), H(q)) and np.array_equal(H(v), H(w))


def test_captured_runs_replay():
    """The run without a workspace under stream capture: every replay, with
    other work between them, continues the trajectory as the eager run does."""
    s = S.solar_system(73, 300 - 31)
    p, v, m = T(s.pos), T(s.vel), T(s.mass)
    lib = C.load()

    def call():
        st = lib.nbody_verlet_run_static(p.data_ptr(), v.data_ptr(), m.data_ptr(), s.n, float(s.G),
                                         float(s.dt), 20, C.NBODY_FP64, 0.0, C.stream_handle(DEV))
        assert st == C.NBODY_OK, C.last_error()

    call()   # (loads the kernels before the capture)
    p.copy_(T(s.pos))
    v.copy_(T(s.vel))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    q, w = T(s.pos), T(s.vel)
    for _ in range(4):
        g.replay()
        nb.verlet_run(q, w, m, s.G, s.dt, 20)
        assert np.array_equal(H(p), H(q)) and np.array_equal(H(v), H(w))


def test_beside_work_that_holds_the_gpu():
    """A run enqueued while force passes over 60,000 bodies occupy the chip on
    another stream equals the run alone, bit for bit."""
    s = S.solar_system(74, 2000 - 31)
    want = run(s, [400])
    big = S.solar_system(75, 60000 - 31)
    bp, bm = T(big.pos), T(big.mass)
    out = torch.empty((3, big.n), dtype=torch.float64, device=DEV)
    p, v, m = T(s.pos), T(s.vel), T(s.mass)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        for _ in range(8):
            nb.accel(bp, bm, big.G, out=out)
    with torch.cuda.stream(b):
        for _ in range(4):
            nb.verlet_run(p, v, m, s.G, s.dt, 100)
    torch.cuda.synchronize()
    assert np.array_equal(H(p), want[0]) and np.array_equal(H(v), want[1])


def ensemble(sizes, seed):
    parts = [S.solar_system(seed + k, n - 11, n_major=10) if n > 11 else
             S.System(*S.random_cluster(seed + k, n)) for k, n in enumerate(sizes)]
    cat = lambda f: np.concatenate([f(x) for x in parts], axis=-1)
    offs = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    return parts, offs, cat(lambda x: x.pos), cat(lambda x: x.vel), cat(lambda x: x.mass)


# one system; sizes on either side of a workgroup's targets; systems spread over
# all XCDs; every shape by total size (1,024, 4,096, 12,288 bodies); one
# workgroup per system; more systems than workgroups fit at once
ENSEMBLES = {
    "one": [900], "tiny": [1, 2, 3, 4, 5, 33], "three": [239, 240, 241],
    "4096": [31, 32, 33, 700, 1000, 1200], "12288": [2048, 2047, 500, 64, 65] + [300] * 12,
    "small-many": [40 + (7 * k) % 361 for k in range(80)],
    "large-many": [300 + (311 * k) % 1749 for k in range(20)],
    "all-whole": [30 + k % 9 for k in range(1300)],
}


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("split", 1e-10)])
@pytest.mark.parametrize("name", list(ENSEMBLES))
def test_ensembles_match_oracle_and_chain(name, precision, tol):
    sizes = ENSEMBLES[name]
    parts, offs, pos, vel, mass = ensemble(sizes, 80)
    G, dt = S.G_AU_DAY_MSUN, 0.1
    runs = []
    for steps in ([9], [4, 1, 4]):
        p, v = T(pos), T(vel)
        for k in steps:
            nb.verlet_run_batched(p, v, T(mass), offs, G, dt, k, precision=precision)
        runs.append((H(p), H(v)))
    assert np.array_equal(runs[0][0], runs[1][0]) and np.array_equal(runs[0][1], runs[1][1])
    for k in {0, len(sizes) // 2, len(sizes) - 1, int(np.argmax(sizes))}:
        a, b = offs[k], offs[k + 1]
        pr, vr = oracle.verlet(parts[k].pos, parts[k].vel, parts[k].mass, G, dt, 9)
        got = runs[0][0][:, a:b]
        assert np.linalg.norm(got - pr) <= tol * np.linalg.norm(pr), (k, sizes[k])


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("split", 2e-12)])
@pytest.mark.parametrize("n", [1280, 1281, 1536, 1537, 2304, 2305, 2560, 2561])
def test_shapes_with_three_and_five_lanes_side_by_side(n, precision, tol):
    test_shapes_match_oracle_and_chain(n, precision, tol)
