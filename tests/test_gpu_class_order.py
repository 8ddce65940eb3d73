"""The split form's class order (heavy bodies first, each class in the original
order) where its launch changes: slices of 1,024 bodies, waves of 64, all,
none and single heavy bodies, ensembles.  Checked through the forces: with
masses that are powers of two the order of a class changes the FP32 sums of
the light bodies, so the split accelerations are compared bit for bit with
those of the same system given in class order already."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"
G = S.G_AU_DAY_MSUN


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def H(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def system(n, heavy, seed):
    """n bodies, the ones with True in `heavy` of mass 1e-6, the others 1e-15."""
    r = np.random.default_rng(seed)
    pos, vel = r.uniform(-3, 3, (3, n)), r.normal(0, 1e-3, (3, n))
    mass = np.where(heavy, 1e-6, 1e-15) * (1 + r.integers(0, 8, n))
    return pos, vel, mass


def patterns(n, r):
    yield "none", np.zeros(n, bool)
    yield "all", np.ones(n, bool)
    yield "last", np.arange(n) == n - 1
    yield "every 63rd", np.arange(n) % 63 == 62
    yield "random", r.random(n) < 0.1


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 5000, 20000])
def test_class_order_of_one_system(n):
    r = np.random.default_rng(n)
    for name, heavy in patterns(n, r):
        pos, vel, mass = system(n, heavy, n)
        order = np.concatenate([np.nonzero(heavy)[0], np.nonzero(~heavy)[0]])
        a = H(nb.accel(T(pos), T(mass), G, precision="split"))
        b = H(nb.accel(T(pos[:, order]), T(mass[order]), G, precision="split"))
        assert np.array_equal(a[:, order], b), (n, name)
        p, v = T(pos), T(vel)
        nb.verlet_run(p, v, T(mass), G, 0.1, 2, precision="split")
        q, w = T(pos[:, order]), T(vel[:, order])
        nb.verlet_run(q, w, T(mass[order]), G, 0.1, 2, precision="split")
        assert np.array_equal(H(p)[:, order], H(q)) and np.array_equal(H(v)[:, order], H(w))


@pytest.mark.parametrize("sizes", [[5, 64, 1, 1024, 1025], [3000, 2500, 10]])
def test_class_order_of_ensembles(sizes):
    offs = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offs[-1])
    r = np.random.default_rng(3)
    for name, heavy in patterns(n, r):
        pos, vel, mass = system(n, heavy, 7)
        order = np.concatenate([a + np.concatenate([np.nonzero(heavy[a:b])[0],
                                                    np.nonzero(~heavy[a:b])[0]])
                                for a, b in zip(offs, offs[1:])])
        p, v = T(pos), T(vel)
        nb.verlet_run_batched(p, v, T(mass), offs.tolist(), G, 0.1, 2, precision="split")
        q, w = T(pos[:, order]), T(vel[:, order])
        nb.verlet_run_batched(q, w, T(mass[order]), offs.tolist(), G, 0.1, 2, precision="split")
        assert np.array_equal(H(p)[:, order], H(q)) and np.array_equal(H(v)[:, order], H(w)), name
