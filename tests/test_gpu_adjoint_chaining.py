"""The reverse sweep works on the forward run's own positions: the gradients do
not depend, bit for bit, on where the checkpoints lie or on whether the
forward run was a call of its own, and its final state is that of a plain run.
At sizes on both sides of the sweep's forms, by default and with the tile of
the product or of the run chosen."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"
STEPS = 23
DT = 4.0   # (days; long, so that a sum of the forces rounded otherwise shows in the positions)


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def check(n):
    s = S.solar_system(n % 19, n - 31)
    r = np.random.default_rng(n)
    lr, lv = T(r.standard_normal((3, n))), T(r.standard_normal((3, n)))
    pos, vel, mass = T(s.pos), T(s.vel), T(s.mass)
    p, v = pos.clone(), vel.clone()
    nb.verlet_run(p, v, mass, s.G, DT, STEPS)
    want = None
    for K in (STEPS, 11, 5):   # one segment; two and a step; ragged
        out = nb.verlet_adjoint(pos, vel, mass, s.G, DT, STEPS, K, lr, lv)
        assert torch.equal(out[3], p) and torch.equal(out[4], v), (n, K)
        want = want or out[:3]
        pT, vT, ck = nb.verlet_checkpoints(pos, vel, mass, s.G, DT, STEPS, K)
        assert torch.equal(pT, p) and torch.equal(vT, v), (n, K)
        two = nb.verlet_adjoint_from_checkpoints(ck, mass, s.G, DT, STEPS, K, lr, lv)
        for a, b, c in zip(want, out, two):
            assert torch.equal(a, b) and torch.equal(a, c), (n, K)


@pytest.mark.parametrize("n", [79, 131, 700, 2079, 2251, 2252, 2560, 2561, 3000, 3073, 4095, 4096])
def test_gradients_do_not_depend_on_the_checkpoints(n):
    nb.reset_caches()
    check(n)


@pytest.mark.parametrize("kind,tile", [(1, (1, 2, 16, 1)), (1, (4, 4, 1, 5)), (0, (1, 2, 4, 1)),
                                       (0, (4, 4, 1, 5))])
@pytest.mark.parametrize("n", [131, 2079, 3000])
def test_gradients_with_a_tile_do_not_depend_on_the_checkpoints(n, kind, tile):
    nb.reset_caches()
    nb.set_tile(kind, "fp64", n, *tile)
    check(n)
    nb.reset_caches()
