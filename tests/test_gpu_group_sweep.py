"""The reverse sweep by workgroups that stay on the chip (80 to 4,095 bodies):
at the sizes where its shape changes, with segments that divide the run or
leave one step over, and longer than one launch, against the sweep by one
product and reduction per position (chosen by setting its tile).

Forward runs and recomputed positions are those of the same kernel on both
sides, so the gradients differ by the rounding of their sums: n terms in another
order, at most n 2^-53 of a sum of magnitudes on each side, over the steps."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def gradients(n, steps, K, per_position):
    nb.reset_caches()
    if per_position:
        nb.set_tile(1, "fp64", n, 1, 2, 16, 1)
    rng = np.random.default_rng(n + steps)
    s = S.solar_system(n % 11, n - 31)
    out = nb.verlet_adjoint(T(s.pos), T(s.vel), T(s.mass), s.G, 0.1, steps, K,
                            T(rng.standard_normal((3, n))), T(rng.standard_normal((3, n))))
    torch.cuda.synchronize()
    nb.reset_caches()
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("n,steps,K", [
    (79, 7, 3), (80, 7, 3), (81, 6, 2), (256, 7, 7), (257, 2, 5), (1024, 9, 4), (1025, 7, 3),
    (2048, 7, 3), (2049, 5, 4), (2560, 7, 3), (2561, 3, 2), (3072, 7, 3), (3073, 4, 4),
    (4095, 7, 3), (4096, 3, 2), (300, 1, 4), (300, 4, 1), (90, 2200, 1100)])
def test_sweep_matches_one_product_per_position(n, steps, K):
    a = gradients(n, steps, K, False)
    b = gradients(n, steps, K, True)
    tol = 2 * (steps + 1) * n * 2.0 ** -53
    for x, y in zip(a[:3], b[:3]):
        assert np.isfinite(x).all()
        assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    assert np.array_equal(a[3], b[3]) and np.array_equal(a[4], b[4])
    for x, y in zip(a, gradients(n, steps, K, False)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [1280, 1281, 1536, 1537])
def test_sweep_with_three_and_five_lanes_side_by_side(n):
    test_sweep_matches_one_product_per_position(n, 7, 3)


@pytest.mark.parametrize("n", [1670, 1671, 2079, 2251, 2252])
@pytest.mark.parametrize("steps,K", [(11, 2), (13, 4)])
def test_sweep_beside_the_recompute_of_many_segments(n, steps, K):
    test_sweep_matches_one_product_per_position(n, steps, K)


def test_two_streams_at_once_equal_one_after_the_other():
    """Two reverse sweeps in flight, each beside its recompute: whichever workgroups
    come late, the gradients are the same bit for bit."""
    n, steps, K = 700, 60, 10
    s = S.solar_system(5, n - 31)
    args = [T(s.pos), T(s.vel), T(s.mass), s.G, 0.1, steps, K, T(np.ones((3, n))),
            T(np.ones((3, n)))]
    one = [x.clone() for x in nb.verlet_adjoint(*args)]
    torch.cuda.synchronize()
    outs = []
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(3):
        for st in streams:
            with torch.cuda.stream(st):
                outs.append(nb.verlet_adjoint(*args))
    torch.cuda.synchronize()
    for o in outs:
        for x, y in zip(one, o):
            assert torch.equal(x, y)
