"""Host logic of bench.py (no GPU): the round kernels' algorithmic bytes where
the first round runs without the color kernel."""
import importlib.util
import os
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_rows_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def stats(color, detect, visits=150, entries=700):
    return SimpleNamespace(color_launches=color, detect_launches=detect, vertex_visits=visits, edge_visits=entries)


def test_color_bytes_leave_out_the_round_without_a_color_launch(bench):
    # 100 vertices and 400 entries in round 1, 50 and 300 in the others
    assert bench.d1_kernel_bytes(stats(4, 5), 100, 400) == \
        (20 * 50 + 8 * 300, 20 * 50 + 8 * 300 + 16 * 100 + 4 * 400)
    assert bench.d1_kernel_bytes(stats(5, 5), 100, 400) == (20 * 150 + 8 * 700,) * 2
    # two hops, mean degree 2: 200 of the 400 are first-hop entries
    later = 20 * 50 + 12 * 100 + 8 * 200
    assert bench.pull_two_hop_bytes(stats(4, 5), 2, 100, 400) == (later, later + 16 * 100 + 12 * 200 + 4 * 200)
    assert bench.pull_two_hop_bytes(stats(5, 5), 2, 100, 400) == (20 * 150 + 12 * 300 + 8 * 400,) * 2
