"""The whole library on the CPU (its sources compiled against the host
emulation of the device operations) against the oracle: every engine, with the
wavefronts of a workgroup in different orders between barriers."""
import ctypes

import numpy as np
import pytest

import emu_lib
import graphgen as gg
import oracle
from paper_2107_00075_amd._binding import COLOR_FLAG_NO_TAIL, ENGINE_INCREMENTAL, ENGINE_PULL, CParams, CStats


@pytest.fixture(scope="module")
def lib():
    lib = emu_lib.load_library()
    yield lib


def run(lib, kind, g, seed, engine, flags=0, init=None, lanes=(0, 0, 0)):
    rows = g
    if kind == "pd2":
        rows = gg.square_pattern_bipartite(g)
        arrays = (rows.row_ptr, rows.col_idx, rows.col_ptr, rows.row_idx)
        sizes = (rows.n_rows, rows.n_cols)
    else:
        arrays = (g.row_ptr, g.col)
        sizes = (g.n,)
    arrays = [np.ascontiguousarray(a, dtype=np.int32) for a in arrays]
    params, st = CParams(), CStats()
    params.engine, params.flags, params.tail_checkin_us = engine, flags, 10_000_000
    params.lanes[:] = lanes
    colors = np.zeros(g.n, np.int32)
    rc = getattr(lib, f"color_{kind}")(*sizes, *map(emu_lib.ptr, arrays), ctypes.c_uint32(seed), None,
                                       emu_lib.ptr(init), emu_lib.ptr(colors), ctypes.byref(st), ctypes.byref(params),
                                       None)
    ref = getattr(oracle, f"color_{kind}")(rows, seed=seed, init=init)
    assert rc == 0
    assert np.array_equal(colors, ref.colors)
    assert (st.rounds, st.vertex_visits, st.edge_visits) == (ref.rounds, ref.vertex_visits, ref.edge_visits)
    return st


GRAPHS = {"er": lambda: gg.erdos_renyi(150, 14.0, 3), "rmat": lambda: gg.rmat(8, 6, seed=2), "star": lambda: gg.star(120),
          "mesh": lambda: gg.stencil((6, 5, 4), 27)}


# every round as its own launches; in the cooperative launches; without lists
@pytest.mark.parametrize("engine,flags", [(ENGINE_INCREMENTAL, COLOR_FLAG_NO_TAIL), (ENGINE_INCREMENTAL, 0),
                                          (ENGINE_PULL, 0)])
@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("kind", ["d1", "d2", "pd2"])
def test_engines(lib, kind, graph, engine, flags):
    g = GRAPHS[graph]()
    full = getattr(oracle, "color_d1" if kind == "d1" else "color_d2")(g, seed=9).colors
    for order in range(3):
        lib.emu_start(0, 8, ctypes.c_uint64(order))
        run(lib, kind, g, 5, engine, flags)
    run(lib, kind, g, 5, engine, flags, init=np.where(np.arange(g.n) % 4 == 0, full, 0).astype(np.int32))


@pytest.mark.parametrize("lanes", [(1, 2, 8), (2, 16, 32), (64, 64, 64)])
def test_lane_groups(lib, lanes):
    lib.emu_start(0, 8, ctypes.c_uint64(7))
    for flags in (0, COLOR_FLAG_NO_TAIL):
        run(lib, "d1", gg.erdos_renyi(400, 10.0, 1), 3, ENGINE_INCREMENTAL, flags, lanes=lanes)
    run(lib, "d1", gg.erdos_renyi(400, 10.0, 1), 3, ENGINE_PULL, lanes=lanes)


def test_tail_kernel_down_to_the_core_kernels(lib):
    lib.emu_start(0, 8, ctypes.c_uint64(3))
    st = run(lib, "d1", gg.erdos_renyi(2500, 16.0, 1), 3, ENGINE_INCREMENTAL)
    assert st.tail_rounds > 0
