"""The neighbourhood walks' source, run on the CPU by the host emulation, on
rows that end at the last entry an int32 offset can name."""
import numpy as np
import pytest

import emu_lib

SCAN, WALK, WORK, SETS = range(4)
D1, D2, PD2 = 1, 2, 3


@pytest.fixture(scope="module")
def lib():
    lib = emu_lib.load("scan_host")
    lib.walk_at_the_end.restype = emu_lib.ctypes.c_int64
    return lib


def check(lib, what, mode, group, length, second):
    n = max(length, length * second)
    seen = np.zeros(n + 1, np.int32)
    got = lib.walk_at_the_end(what, mode, group, length, second, emu_lib.ptr(seen))
    assert got >= 0, "the walk died"
    ref = np.zeros(n + 1, np.int32)
    if mode != PD2:
        ref[:length] += 1
    if mode != D1:
        ref[:length * second] += 1
    if what == WORK:
        assert got == length * (1 + second)
    else:
        assert np.array_equal(seen, np.minimum(ref, 1) if what == SETS else ref)


@pytest.mark.parametrize("length", [1, 7, 100, 3000])
@pytest.mark.parametrize("group", [1, 4, 64, 256])
def test_scan(lib, group, length):
    check(lib, SCAN, D1, group, length, 0)
    for second in (0, 1, 3, 4, 9):
        check(lib, SCAN, D2, group, length, second)
        check(lib, SCAN, PD2, group, length, second)


@pytest.mark.parametrize("length", [1, 15, 17, 130])
@pytest.mark.parametrize("group", [16, 64])
def test_two_hop_walk(lib, group, length):
    for second in (0, 1, 5, 40):
        check(lib, WALK, D2, group, length, second)
        check(lib, WALK, PD2, group, length, second)


@pytest.mark.parametrize("length", [1, 16, 300, 5000])
@pytest.mark.parametrize("group", [1, 64, 256])
def test_work(lib, group, length):
    check(lib, WORK, PD2, group, length, 3)


@pytest.mark.parametrize("length", [1, 1000, 5000])
def test_sets(lib, length):
    check(lib, SETS, D2, 0, length, 3)
    check(lib, SETS, PD2, 0, length, 3)
