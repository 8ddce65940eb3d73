"""nbody_set_tuned_tile takes and refuses what nbody_set_tile does, and
nbody_get_tile reports what either entered."""
import ctypes

import pytest

from paper_2112_15079_amd import _capi as C


@pytest.mark.parametrize("kind,precision,n,tile", [
    (0, 0, 10425, (4, 2, 7, 0)), (0, 0, 10425, (1, 2, 9, 3)), (0, 0, 400, (1, 16, 2, 3)),
    (0, 0, 513, (1, 16, 1, 3)), (0, 0, 3000, (2, 8, 1, 4)), (1, 0, 3000, (1, 2, 1, 4)),
    (1, 0, 100, (1, 1, 1, 1)), (1, 0, 100, (4, 1, 1, 0)), (1, 0, 131073, (2, 4, 1, 5)),
    (2, 0, 0, (2, 1, 16, 1)), (2, 0, 0, (1, 16, 4, 3)), (3, 0, 10, (1, 1, 1, 0)),
    (0, 7, 100, (1, 1, 1, 0)), (0, 2, 10425, (2, 4, 1, 5)), (0, 2, 10425, (1, 1, 1, 0)),
    (0, 0, 0, (1, 1, 1, 0)), (0, 0, 10425, (1, 1, 65, 0))])
def test_takes_and_refuses_what_set_tile_does(kind, precision, n, tile):
    lib = C.load()
    got = []
    for call in (lib.nbody_set_tile, lib.nbody_set_tuned_tile):
        lib.nbody_reset_caches()
        t = C.Tile()
        st = call(kind, precision, n, ctypes.byref(C.Tile(*tile)))
        got.append((st, C.last_error() if st else "",
                    lib.nbody_get_tile(kind, precision, n, ctypes.byref(t)), t.as_dict()))
    lib.nbody_reset_caches()
    assert got[0] == got[1]
    assert lib.nbody_set_tuned_tile(0, 0, 10, None) == C.NBODY_EINVAL
