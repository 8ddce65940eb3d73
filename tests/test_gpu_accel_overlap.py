"""Accelerations stored over the positions (or masses) they were computed from:
every kernel that reads and stores in one launch has to go by way of the
workspace, so the result is that of a separate output bit for bit.  Sizes on
each side of the kernels' limits; a tile that fuses pass and step; outputs that
overlap the positions in part and the masses in full."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def check(n, precision):
    s = S.solar_system(n % 17, n - 31)
    pos, mass = T(s.pos), T(s.mass)
    want = nb.accel(pos, mass, s.G, precision=precision)
    for _ in range(3):
        p = pos.clone()
        assert nb.accel(p, mass, s.G, precision=precision, out=p) is p
        assert torch.equal(p, want), n
        buf = torch.cat([pos, mass[None]])   # x, y, z, m: the output over y, z and m
        nb.accel(buf[:3], buf[3], s.G, precision=precision, out=buf[1:])
        assert torch.equal(buf[1:], want) and torch.equal(buf[0], pos[0]), n


@pytest.mark.parametrize("precision", ["fp64", "split"])
@pytest.mark.parametrize("n", [79, 80, 131, 300, 512, 513, 1000, 2079, 4000, 4095, 4096])
def test_accelerations_over_their_inputs(n, precision):
    nb.reset_caches()
    check(n, precision)


@pytest.mark.parametrize("n,tile", [(300, (1, 8, 1, 4)), (3000, (2, 8, 1, 4)), (131, (1, 16, 7, 3)),
                                    (1000, (1, 2, 8, 1))])
def test_accelerations_over_their_inputs_with_a_tile(n, tile):
    nb.reset_caches()
    nb.set_tile(0, "fp64", n, *tile)
    check(n, "fp64")
    nb.reset_caches()
