"""The core kernels' source, run on the CPU by the host emulation of the
device operations, against the oracle."""
import numpy as np
import pytest

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
