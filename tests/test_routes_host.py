"""The table of routes (launches or the persistent launch) beside the tunings."""
import ctypes as C

import pytest

from paper_2205_04295_amd import _abi, tune


@pytest.fixture(autouse=True)
def _restore():
    saved = {(N, c): tune.get_tuning(N, c, M=3) for N in (128, 256) for c in (0, 1)}
    yield
    for (N, c), t in saved.items():
        tune.set_tuning(N, c, **t)


def test_set_tuning_sets_the_route():
    assert tune.get_route(256, 0, M=3) == "auto"
    default = tune.get_tuning(256, 0, M=3)
    tune.set_tuning(256, 0, M=3, **dict(default, cols_radix=4))
    assert tune.get_route(256, 0, M=4) == "launches"      # the mode class of 3 and 4
    assert tune.get_route(256, 0, M=5) == "auto" and tune.get_route(256, 1, M=3) == "auto"
    tune.set_tuning(256, 0, M=3, **default)               # what a program restores
    assert tune.get_route(256, 0, M=3) == "auto"


def test_route_round_trip_and_errors():
    tune.set_route(128, 1, "persistent")
    assert [tune.get_route(128, 1, M=m) for m in (1, 2, 3, 8)] == ["persistent"] * 4
    assert tune.get_route(128, 0) == "auto"
    tune.set_route(128, 1, "launches", M=2)
    assert tune.get_route(128, 1, M=2) == "launches" and tune.get_route(128, 1, M=3) == "persistent"
    # a tuning and its route, saved and restored
    t, r = tune.get_tuning(128, 1, M=3), tune.get_route(128, 1, M=3)
    tune.set_tuning(128, 1, M=3, **dict(t, rows_threads=512))
    assert tune.get_route(128, 1, M=3) == "launches"
    tune.set_tuning(128, 1, M=3, **t)
    tune.set_route(128, 1, r, M=3)
    assert tune.get_route(128, 1, M=3) == "persistent"
    lib, out = _abi.load(), C.c_int32(0)
    assert lib.mrpie_set_route(100, 0, 0, 1) == _abi.MRPIE_EUNSUPPORTED
    assert lib.mrpie_set_route(128, 9, 0, 1) == lib.mrpie_set_route(128, 0, 3, 1) == _abi.MRPIE_EINVAL
    assert lib.mrpie_set_route(128, 0, 0, 3) == lib.mrpie_set_route(128, 0, 0, -1) == _abi.MRPIE_EINVAL
    assert lib.mrpie_get_route(128, 0, 0, C.byref(out)) == lib.mrpie_get_route(128, 1, 0, None) == _abi.MRPIE_EINVAL
