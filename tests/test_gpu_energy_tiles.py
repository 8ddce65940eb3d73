"""The energy kernels' tiles (256 rows, 128 sources): sizes around their edges,
massless and coincident-free extremes, against the oracle.  Each side adds
compensated sums of terms with a relative error of a few rounding units, so
1e-14 of the sum of magnitudes holds with a wide margin."""
import numpy as np
import pytest
import torch

import oracle
import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 255, 256, 257, 384, 385, 1025, 5000])
def test_energy_and_momenta_at_tile_edges(n):
    pos, vel, mass = S.random_cluster(n, n, spread=2.0)
    mass[::5] = 0.0
    G = 1.7
    e = nb.energy(T(pos), T(vel), T(mass), G).cpu().numpy()
    ref = np.array(oracle.energy(pos, vel, mass, G))
    assert np.all(np.abs(e - ref) <= 1e-14 * np.abs(ref[:2]).sum())
    m = nb.momenta(T(pos), T(vel), T(mass)).cpu().numpy()
    P = (mass * vel).sum(1)
    L = (mass * np.cross(pos.T, vel.T).T).sum(1)
    bound = 1e-14 * (mass * np.linalg.norm(vel, axis=0) * (1 + np.linalg.norm(pos, axis=0))).sum()
    assert np.all(np.abs(m - np.concatenate([P, L])) <= bound)
