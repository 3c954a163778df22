"""The benchmark's bytes per site follow the library's own rule for two steps in
one launch, which lb_step_launches reports (host only)."""

import ctypes

import pytest

import bench
from paper_1703_00186_amd import lb as lbmod


def launches(n, lx, ly, precision="fp64", ybc="walls", layout="column", **par):
    return lbmod.step_launches(lbmod.make_lattice(lx, ly, precision, ybc, layout),
                               lbmod.make_params(**par), n)


@pytest.mark.parametrize("lattice,pairs", [
    (dict(lx=1920, ly=2048), True),
    (dict(lx=20000, ly=56), False),  # two waves of 52 rows against one of 56
    (dict(lx=64, ly=48), True),      # fewer than 128 columns of windows
    (dict(lx=256, ly=128), False),
    (dict(lx=1920, ly=2048, precision="fp32s"), True),
    (dict(lx=1920, ly=2048, precision="fp32s", layout="soa"), False),
    (dict(lx=14003, ly=40, precision="fp32s"), False),  # windows less than 3/4 full
    (dict(lx=1920, ly=2048, precision="fp32l"), False),
    (dict(lx=1024, ly=1000, regularize=0), True),
    (dict(lx=1024, ly=1000, regularize=0, layout="soa"), False),
    (dict(lx=1920, ly=2048, kernel="split"), False),
    (dict(lx=1920, ly=2048, check_finite=5), False),
])
def test_launches_of_a_run(lattice, pairs):
    for n, two in ((0, 0), (1, 1), (4, 4), (5, 3), (8, 6), (9, 5), (20, 12), (21, 11)):
        assert launches(n, **lattice) == (two if pairs else n), n


def test_bytes_follow_the_launches():
    assert bench.moved_bytes_per_site("fp64", 1920, 2048, 20) == 240 * 12 / 20
    assert bench.moved_bytes_per_site("fp64", 20000, 56, 20) == 240
    assert bench.moved_bytes_per_site("fp64", 64, 48, 20) == 240 * 12 / 20
    assert bench.moved_bytes_per_site("fp32s", 1920, 2048, 200) == 296 * 102 / 200
    assert bench.moved_bytes_per_site("fp32s", 1920, 2048, 200, layout="soa") == 296
    assert bench.moved_bytes_per_site("fp32c", 1920, 2048, 200) == 304


def test_arguments():
    lib = lbmod.load_library()
    lat, par = lbmod.make_lattice(64, 48), lbmod.make_params()
    out = ctypes.c_int(0)
    assert lib.lb_step_launches(ctypes.byref(lat), ctypes.byref(par), -1, ctypes.byref(out)) == -1
    assert lib.lb_step_launches(ctypes.byref(lat), ctypes.byref(par), 1, None) == -1
    assert lib.lb_step_launches(None, ctypes.byref(par), 1, ctypes.byref(out)) == -1
    lat.lx = 3
    assert lib.lb_step_launches(ctypes.byref(lat), ctypes.byref(par), 1, ctypes.byref(out)) == -1
