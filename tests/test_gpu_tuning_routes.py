"""A tuning file has the effect that the autotuner had in the process that wrote
it: after load_tuning() runs, gradients and ensembles take the kernels that
they took after the autotuner (and so its speed), bit for bit."""
import numpy as np
import pytest
import torch

import solar_ics as S

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")

DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def after_autotune_and_after_load(tune, work, path):
    nb.reset_caches()
    tune()
    tuned = work()
    nb.save_tuning(path)
    nb.reset_caches()
    assert nb.load_tuning(path) == 1
    loaded = work()
    nb.reset_caches()
    assert all(torch.equal(a, b) for a, b in zip(tuned, loaded))


# (a long step, so that forces summed in another order show in the positions)
@pytest.mark.parametrize("precision", ["fp64", "split"])
@pytest.mark.parametrize("n", [60, 131, 1000, 4200])
def test_runs(n, precision, tmp_path):
    s = S.solar_system(3, n - 31)
    pos, vel, mass = T(s.pos), T(s.vel), T(s.mass)

    def work():
        p, v = pos.clone(), vel.clone()
        nb.verlet_run(p, v, mass, s.G, 4.0, 40, precision=precision)
        return p, v, nb.accel(pos, mass, s.G, precision=precision)

    after_autotune_and_after_load(lambda: nb.autotune(pos, mass, s.G, precision=precision), work,
                                  str(tmp_path / "tuning.json"))


@pytest.mark.parametrize("n", [131, 1000])
def test_gradients(n, tmp_path):
    s = S.solar_system(4, n - 31)
    pos, vel, mass = T(s.pos), T(s.vel), T(s.mass)
    g = T(np.random.default_rng(1).standard_normal((3, n)))
    after_autotune_and_after_load(
        lambda: nb.autotune(pos, mass, s.G, kind=1),
        lambda: nb.verlet_adjoint(pos, vel, mass, s.G, 4.0, 20, 7, g, g),
        str(tmp_path / "tuning.json"))


def test_ensembles(tmp_path):
    sizes = [200, 37, 120, 64, 333]
    offs = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    parts = [S.solar_system(k, n - 31) for k, n in enumerate(sizes)]
    pos, vel, mass = (T(np.concatenate([getattr(x, f) for x in parts], axis=-1))
                      for f in ("pos", "vel", "mass"))
    G = S.G_AU_DAY_MSUN

    def work():
        p, v = pos.clone(), vel.clone()
        nb.verlet_run_batched(p, v, mass, offs, G, 4.0, 40)
        return p, v

    after_autotune_and_after_load(lambda: nb.autotune_batched(pos, mass, offs, G), work,
                                  str(tmp_path / "tuning.json"))
