"""The each-pair-once FP64 pass in quarters of a range pair (up to 19 ranges of
256 bodies): one range, ragged last ranges and blocks, the last size that takes
it and the first that does not, in an evaluation and in a run, against the
oracle at the tolerance of the other force passes."""
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


def rel(a, b):
    return float(np.max(np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)))


@pytest.mark.parametrize("n", [33, 64, 65, 256, 257, 321, 511, 512, 513, 1000, 4095, 4096, 4097,
                               4609, 4864, 4865])
def test_quarters_match_oracle(n):
    nb.reset_caches()
    nb.set_tile(0, "fp64", n, 4, 4, 1, 5)
    s = S.solar_system(n % 13, n - 31)
    p, v, m = T(s.pos), T(s.vel), T(s.mass)
    a = nb.accel(p, m, s.G)
    b = nb.accel(p, m, s.G)
    nb.verlet_run(p, v, m, s.G, s.dt, 3)
    torch.cuda.synchronize()
    nb.reset_caches()
    assert torch.equal(a, b)
    assert rel(a.cpu().numpy(), oracle.accel(s.pos, s.mass, s.G)) <= 1e-13
    pr, vr = oracle.verlet(s.pos, s.vel, s.mass, s.G, s.dt, 3)
    assert rel(p.cpu().numpy()[:, 1:], pr[:, 1:]) <= 1e-12
    assert rel(v.cpu().numpy()[:, 1:], vr[:, 1:]) <= 1e-12
