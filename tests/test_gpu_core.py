"""The core kernels (the last rounds on rows of adjacency bits) against the
oracle: worklists at the edges of each stage's capacity, tentative colors
spread wider than the color slots, colors beyond the forbidden-color window,
round caps inside each stage, and every key."""
import numpy as np
import pytest

import graphgen as gg
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


def check(gc, g, seed, kind="d1", flags=0, prio=None, init=None, max_rounds=0):
    """The coloring with every round inside the tail and core kernels equals the oracle's."""
    ref = getattr(oracle, f"color_{kind}")(g, seed=seed, prio=prio, init=init, max_rounds=max_rounds,
                                           recolor_degrees=bool(flags & gc.COLOR_FLAG_RECOLOR_DEGREES))
    got, st = getattr(gc, f"color_{kind}")(
        dev(g.row_ptr), dev(g.col), seed=seed, trace_cap=4096, allow_partial=max_rounds > 0,
        prio=None if prio is None else torch.from_numpy(prio.view(np.int32)).cuda(),
        init_colors=None if init is None else dev(init),
        params=gc.Params(engine=gc.ENGINE_INCREMENTAL, tail_threshold=1 << 30, max_rounds=max_rounds, flags=flags))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert st.rounds == ref.rounds == st.tail_rounds and st.worklist == ref.worklist[:4096]
    assert st.num_colors == int(ref.colors.max())
    assert st.vertex_visits == ref.vertex_visits and st.edge_visits == ref.edge_visits
    assert st.converged == ref.converged
    return st


# one workgroup: up to 1024 vertices; 64-vertex workgroups up to 4096, then
# to 16384; 96-vertex workgroups up to 24576; above, the tail kernel first
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4096, 4097, 16384, 16385, 24576, 24577])
def test_core_sizes(gc, n):
    g = gg.erdos_renyi(n, min(24.0, n / 2), n) if n > 2 else gg.path(n)
    check(gc, g, 3)


@pytest.mark.parametrize("n", [700, 1500, 5000])
def test_core_colors_beyond_the_window(gc, n):
    """Dense graphs: far more than 64 colors are taken inside one launch."""
    rng = np.random.default_rng(n)
    g = gg.complete(n) if n < 2000 else gg.random_small_graph(n, 0.2, rng)
    st = check(gc, g, 5)
    assert st.num_colors > 130


def ladder(m, steps, seed):
    """m uncolored vertices in a sparse random graph; vertex i is also joined
    to the committed vertices of colors 1 .. k_i, k_i spread over 0 .. steps."""
    rng = np.random.default_rng(seed)
    k = rng.integers(0, steps + 1, m)
    i = np.repeat(np.arange(m), k)
    j = np.concatenate([np.arange(x) for x in k]) if k.sum() else np.zeros(0, np.int64)
    u = rng.integers(0, m, 6 * m)
    v = rng.integers(0, m, 6 * m)
    g = gg.csr_from_pairs(m + steps, np.concatenate([i, u]), np.concatenate([j + m, v]))
    init = np.zeros(m + steps, np.int32)
    init[m:] = np.arange(1, steps + 1)
    return g, init


@pytest.mark.parametrize("m", [50, 1024, 1025, 3000, 9000, 20000])
@pytest.mark.parametrize("steps", [20, 31, 33, 150])
def test_core_spread_tentative_colors(gc, m, steps):
    """Tentative colors spread over more colors than there are slots: the
    one-workgroup stage compares them one by one, the others give the rounds
    back to the tail kernel."""
    g, init = ladder(m, steps, m + steps)
    check(gc, g, 9, init=init)


@pytest.mark.parametrize("cap", [1, 2, 3, 30, 60, 90])
def test_core_round_cap(gc, cap):
    g = gg.rmat(14, 16, seed=3)  # 74 rounds through all three stages
    check(gc, g, 1, max_rounds=cap)


@pytest.mark.parametrize("n", [900, 3000, 12000])
@pytest.mark.parametrize("key", ["degrees", "prio", "prio_ties"])
def test_core_keys(gc, n, key):
    g = gg.erdos_renyi(n, 40.0, n)
    if key == "degrees":
        check(gc, g, 4, flags=gc.COLOR_FLAG_RECOLOR_DEGREES)
        return
    rng = np.random.default_rng(n)
    hi = 1 << 32 if key == "prio" else 7
    check(gc, g, 4, prio=rng.integers(0, hi, n, dtype=np.uint32))


def test_core_two_hop(gc):
    check(gc, gg.erdos_renyi(6000, 16.0, 2), 8, kind="d2")
    check(gc, gg.stencil((23, 19, 17), 27), 8, kind="d2")
