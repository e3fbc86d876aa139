"""Host logic of bench.py (no GPU): the round kernels' algorithmic bytes where
the first round runs without the color kernel, and the counter figures of
kernels with several variants and of the cooperative rounds."""
import importlib.util
import json
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


def test_traffic_of_kernel_variants_and_of_the_cooperative_rounds(bench, tmp_path, monkeypatch):
    from paper_2107_00075_amd.build import source_hash
    kernels = {"detect_round_kernel<1, false>": (27, 100), "detect_round_kernel<1, true>": (1, 380),
               "detect_round_kernel<2, true>": (1, 7), "color_round_kernel<D1>": (27, 50), "inc_tail_kernel": (1, 1000),
               "core_rank_kernel<false>": (1, 10), "core_build_kernel": (1, 200),
               "core_wide_kernel<3, 12, 512>": (1, 30), "core_kernel": (1, 4)}
    path = tmp_path / "traffic.json"
    path.write_text(json.dumps({"source_hash": source_hash(), "workload": "d1", "kernels": {
        k: {"dispatches": n, "hbm_bytes_per_launch": b} for k, (n, b) in kernels.items()}}))
    monkeypatch.setattr(bench, "traffic_file", lambda w: str(path))
    assert bench.load_traffic("detect_round_kernel<D1>", "d1") == (27 * 100 + 380) // 28
    assert bench.load_traffic("detect_round_kernel<D2>", "d1") == 7
    assert bench.load_traffic("detect_round_kernel<PD2>", "d1") is None
    assert bench.load_traffic("color_round_kernel<D1>", "d1") == 50
    assert bench.load_traffic(bench.TAIL_ROUNDS, "d1") == 1000 + 10 + 200 + 30 + 4
    rows = bench.kernel_rows(None, SimpleNamespace(color_kernel_ns=1, color_launches=27, detect_kernel_ns=2,
                                                   detect_launches=28, tail_rounds=5, tail_bytes=9,
                                                   tail_kernel_ns=3),
                             ("color_round_kernel<D1>", "detect_round_kernel<D1>"), 10, 20)
    rate = bench.counter_rate({r[0]: r[1:] for r in rows}, "d1")
    assert rate["bytes"] == 27 * 50 + 28 * ((27 * 100 + 380) // 28) + 1244


@pytest.mark.parametrize("workload", ["d1", "d2pd2"])
def test_committed_summary_names_every_timed_kernel(bench, workload):
    """The committed counter summary holds every round kernel bench.py times."""
    with open(bench.traffic_file(workload)) as f:
        names = json.load(f)["kernels"]
    mode = "D1" if workload == "d1" else "D2"
    for kernel in (f"color_round_kernel<{mode}>", f"detect_round_kernel<{mode}>", "inc_color_kernel",
                   "inc_detect_kernel", bench.TAIL_ROUNDS):
        assert bench.summary_names(kernel, names), kernel
