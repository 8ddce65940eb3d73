"""The split form's class order over more systems than a grid's second and third
dimensions take (65,535), and where many systems share the slices of a large
one."""
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


@pytest.mark.parametrize("sizes", [[2] * 65535, [2] * 65536, [1, 3] * 35000,
                                   [6000] + [3] * 300, [3] * 20000 + [6000]],
                         ids=["65535", "65536", "70000", "301", "20001"])
def test_many_systems(sizes):
    offs = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offs[-1])
    r = np.random.default_rng(n)
    pos, vel = r.uniform(-3, 3, (3, n)), r.normal(0, 1e-3, (3, n))
    mass = np.where(r.random(n) < 0.5, 1e-4, 1e-15) * r.uniform(1, 2, n)
    p, v = T(pos), T(vel)
    nb.verlet_run_batched(p, v, T(mass), offs.tolist(), S.G_AU_DAY_MSUN, 0.1, 3,
                          precision="split")
    got = p.cpu().numpy()
    assert np.isfinite(got).all()
    pick = {0, 1, len(sizes) // 2, len(sizes) - 2, len(sizes) - 1, *range(65530, len(sizes), 997)}
    for k in pick:
        a, b = offs[k], offs[k + 1]
        want, _ = oracle.verlet(pos[:, a:b], vel[:, a:b], mass[a:b], S.G_AU_DAY_MSUN, 0.1, 3)
        assert np.linalg.norm(got[:, a:b] - want) <= 1e-10 * np.linalg.norm(want), k
