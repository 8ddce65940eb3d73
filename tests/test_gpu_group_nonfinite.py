"""Runs, ensembles and gradients that stay on the chip with numbers that are not
finite, the exchange's own sentinel pattern among them: they end, set the
flag, and spread over the bodies as they do by launches (chosen by setting the
tile); other systems of an ensemble are untouched."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"
SENTINEL = np.array([0xFFF4B0D1E5A11CED], dtype=np.uint64).view(np.float64)[0]
BAD = {"nan": np.nan, "inf": np.inf, "sentinel": SENTINEL}
TILE = (1, 2, 4, 1)


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def spoiled(n, what, bad):
    s = S.solar_system(5, n - 31)
    x = {"pos": s.pos.copy(), "vel": s.vel.copy(), "mass": s.mass.copy()}
    x[what][..., n // 3] = bad
    return T(x["pos"]), T(x["vel"]), T(x["mass"])


def run(n, what, bad, precision):
    p, v, m = spoiled(n, what, bad)
    nb.get_flags(clear=True)
    nb.verlet_run(p, v, m, S.G_AU_DAY_MSUN, 0.1, 7, precision=precision)
    flag = nb.get_flags(clear=True)
    return p, v, flag


@pytest.mark.parametrize("precision", ["fp64", "split"])
@pytest.mark.parametrize("name", list(BAD))
@pytest.mark.parametrize("what", ["pos", "vel", "mass"])
@pytest.mark.parametrize("n", [131, 1000, 3000])
def test_runs(n, what, name, precision):
    nb.reset_caches()
    p, v, flag = run(n, what, BAD[name], precision)
    nb.set_tile(0, precision, n, *TILE)
    q, w, by_launches = run(n, what, BAD[name], precision)
    nb.reset_caches()
    assert flag & 1 and by_launches & 1
    assert torch.equal(torch.isfinite(p), torch.isfinite(q))
    assert torch.equal(torch.isfinite(v), torch.isfinite(w))


@pytest.mark.parametrize("name", list(BAD))
def test_ensembles(name):
    sizes = [200, 37, 500, 64]
    offs = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    parts = [S.solar_system(k, n - 31) for k, n in enumerate(sizes)]
    cat = lambda f: np.concatenate([getattr(x, f) for x in parts], axis=-1)
    pos = cat("pos")
    out = []
    for bad in (None, BAD[name]):
        if bad is not None:
            pos[1, 210] = bad   # in the second system
        p, v = T(pos), T(cat("vel"))
        nb.get_flags(clear=True)
        nb.verlet_run_batched(p, v, T(cat("mass")), offs, S.G_AU_DAY_MSUN, 0.1, 7)
        out.append((p, v, nb.get_flags(clear=True)))
    assert out[0][2] == 0 and out[1][2] & 1
    for a, b in zip(out[0][:2], out[1][:2]):
        assert torch.isfinite(a).all() and not torch.isfinite(b[:, 200:237]).any()
        assert torch.equal(a[:, :200], b[:, :200]) and torch.equal(a[:, 237:], b[:, 237:])


@pytest.mark.parametrize("name", list(BAD))
@pytest.mark.parametrize("what", ["pos", "mass", "cotangent"])
@pytest.mark.parametrize("n", [131, 700, 2500])
def test_gradients_end(n, what, name):
    nb.reset_caches()
    p, v, m = spoiled(n, what if what != "cotangent" else "pos",
                      BAD[name] if what != "cotangent" else 1.0)
    g = np.ones((3, n))
    if what == "cotangent":
        g[:, 7] = BAD[name]
    out = nb.verlet_adjoint(p, v, m, S.G_AU_DAY_MSUN, 0.1, 7, 3, T(np.ones((3, n))), T(g))
    torch.cuda.synchronize()
    assert not all(torch.isfinite(x).all() for x in out[:3])
