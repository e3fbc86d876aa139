"""The core kernels against the oracle on graphs whose largest tentative color
falls while vertices that have to climb past it are left."""
import numpy as np
import pytest

import core_cases
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_00075_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def check(gc, g, seed=1, prio=None, init=None, engine=2):
    ref = oracle.color_d1(g, seed=seed, prio=prio, init=init)
    got, st = gc.color_d1(dev(g.row_ptr), dev(g.col), seed=seed, trace_cap=4096,
                          prio=None if prio is None else torch.from_numpy(prio.view(np.int32)).cuda(),
                          init_colors=None if init is None else dev(init), params=gc.Params(engine=engine))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert st.engine == gc.ENGINE_INCREMENTAL
    assert (st.rounds, st.worklist) == (ref.rounds, ref.worklist[:4096])


@pytest.mark.parametrize("path,top,low", core_cases.CLIMBS)
def test_climb(gc, path, top, low):
    g, prio = core_cases.climb(path, top, low)
    check(gc, g, prio=prio)
    # by the library's own choice of the engine, and with the default key
    check(gc, core_cases.climb_by_hash(path, top, low, 3000, 1), engine=gc.ENGINE_AUTO)


# the stage reached from 64 and from 256 workgroups, and from the tail kernel
@pytest.mark.parametrize("n", [1400, 3900, 6000, 24000, 40000])
@pytest.mark.parametrize("path,top,low", [(60, 30, 40), (60, 12, 15)])
def test_climb_beside_a_random_graph(gc, path, top, low, n):
    g, prio = core_cases.beside(*core_cases.climb(path, top, low), n, 2)
    check(gc, g, prio=prio)


def test_five_vertices(gc):
    g, init, prio = core_cases.five()
    check(gc, g, init=init, prio=prio)


# (1500, 0.05, 20): by hand-over
@pytest.mark.parametrize("m,p,steps", core_cases.ANCHORED + [(1500, 0.05, 20)])
def test_dense_with_uneven_forbidden_colors(gc, m, p, steps):
    for seed in range(4):
        g, init = core_cases.anchored(m, p, 0.3, steps, seed)
        check(gc, g, init=init)
