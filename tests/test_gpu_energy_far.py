"""Energies of bodies anywhere: no place in space is the kernels' own (a tile's
missing sources were once massless bodies at 1e18 in each coordinate, and a
body there, or so far away that its distance from there overflows, made the
energy NaN)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.mark.parametrize("n", [2, 3, 127, 129, 300, 1025])
@pytest.mark.parametrize("centre,spread", [(1e18, 0.0), (1e18, 1e16), (1e160, 1e150), (-3e18, 1e17)])
def test_energy_far_from_the_origin(n, centre, spread):
    r = np.random.default_rng(n)
    pos = centre + spread * r.uniform(-1, 1, (3, n)) if spread else 1e18 * r.uniform(-1, 1, (3, n))
    pos[:, 0] = centre
    vel, mass = r.normal(0, 1e-3, (3, n)), r.uniform(1, 2, n)
    ref = np.array(oracle.energy(pos, vel, mass, 2.0))
    assert np.isfinite(ref).all()
    e = nb.energy(T(pos), T(vel), T(mass), 2.0).cpu().numpy()
    assert np.all(np.abs(e - ref) <= 1e-14 * np.abs(ref[:2]).sum())
