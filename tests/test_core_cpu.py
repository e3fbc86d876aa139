"""The core kernels' source, run on the CPU by the host emulation of the
device operations, against the oracle.  The emulation runs the wavefronts of a
workgroup in any order between two barriers, which no run on the device can be
made to do."""
import numpy as np
import pytest

import core_cases
import emu_lib
import graphgen as gg
import oracle


@pytest.fixture(scope="module")
def lib():
    return emu_lib.load("core_host")


def check(lib, g, seed=1, prio=None, init=None, max_rounds=0, order=1):
    ref = oracle.color_d1(g, seed=seed, prio=prio, init=init, max_rounds=max_rounds)
    colors, rounds, visits, left = emu_lib.core_run(lib, g, seed, prio, init, max_rounds, order)
    assert np.array_equal(colors, ref.colors)
    assert (rounds, visits, left) == (ref.rounds, ref.vertex_visits, 0 if ref.converged else 1)


# the 64-workgroup stage, and its rows' hand-over to the one-workgroup stage
@pytest.mark.parametrize("n", [1025, 1500])
def test_hand_over(lib, n):
    check(lib, gg.erdos_renyi(n, 24.0, n), 3, order=0)


# one wavefront to all sixteen of the one-workgroup stage, and the stage before
@pytest.mark.parametrize("n", [64, 65, 300, 1024, 1025])
@pytest.mark.parametrize("order", [0, 1, 2, 3, 4, 5])
def test_wavefront_orders(lib, n, order):
    check(lib, gg.erdos_renyi(n, 24.0, n), 3, order=order)


@pytest.mark.parametrize("cap", [1, 4, 9])
def test_round_cap_in_any_order(lib, cap):
    for order in range(4):
        check(lib, gg.erdos_renyi(700, 24.0, 7), 3, max_rounds=cap, order=order)


@pytest.mark.parametrize("path,top,low", core_cases.CLIMBS)
def test_colors_above_the_active_ones(lib, path, top, low):
    """A color that was committed while the active vertices' colors reached it
    is still there when they have fallen below it and climb past it."""
    g, prio = core_cases.climb(path, top, low)
    check(lib, g, prio=prio)
    check(lib, core_cases.climb_by_hash(path, top, low, 200, 1), seed=1)


@pytest.mark.parametrize("path,top,low", [(60, 30, 40), (60, 12, 15)])
def test_colors_above_the_active_ones_after_a_hand_over(lib, path, top, low):
    g, prio = core_cases.beside(*core_cases.climb(path, top, low), 1400, 2)
    check(lib, g, prio=prio)


def test_five_vertices(lib):
    g, init, prio = core_cases.five()
    check(lib, g, init=init, prio=prio)


@pytest.mark.parametrize("m,p,steps", core_cases.ANCHORED)
def test_dense_with_uneven_forbidden_colors(lib, m, p, steps):
    for seed in range(6 if m < 500 else 1):
        g, init = core_cases.anchored(m, p, 0.3, steps, seed)
        check(lib, g, init=init, order=seed)


@pytest.mark.parametrize("err", [0x800, 0x900])
def test_second_launch_after_the_first(lib, err):
    """After a first launch in which a wait gave up (0x100), what it handed
    over is not complete: the second launch does nothing."""
    colors = np.zeros(100, np.int32)
    assert lib.core_second_launch(100, err, emu_lib.ptr(colors)) == err
    assert (colors == (0 if err & 0x100 else 1)).all()
