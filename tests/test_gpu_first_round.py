"""The pull engine's first round from no colors (no tentative colors are
gathered) and the workgroup's buffer of losers, against the oracle: every bin
kind, worklists around the buffer's size on one workgroup, initial colors
(which take the general round), and every graph kind."""
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


# all light; light and workgroup bins; split vertices as well
BINS = {"light": (0, 0, 0, 0), "block": (4, 8, 12, 0), "split": (2, 4, 8, 16)}


@pytest.mark.parametrize("bins", BINS)
@pytest.mark.parametrize("n, groups", [(767, 1), (1025, 1), (6000, 8)])
@pytest.mark.parametrize("kind", ["d1", "d2", "pd2", "d1 init"])
def test_first_round(gc, kind, n, groups, bins):
    g = gg.erdos_renyi(n, 10, n)
    p = gc.Params(engine=gc.ENGINE_PULL, max_workgroups=groups, bin_hi=BINS[bins])
    kw = dict(seed=2, trace_cap=4096, params=p)
    if kind == "pd2":
        b = gg.square_pattern_bipartite(g)
        ref = oracle.color_pd2(b, seed=2)
        got, st = gc.color_pd2(dev(b.row_ptr), dev(b.col_idx), dev(b.col_ptr), dev(b.row_idx), **kw)
    elif kind == "d2":
        ref = oracle.color_d2(g, seed=2)
        got, st = gc.color_d2(dev(g.row_ptr), dev(g.col), **kw)
    else:
        init = None
        if kind == "d1 init":  # a few vertices keep the colors of a full coloring
            full = oracle.color_d1(g, seed=7).colors
            init = np.where(np.random.default_rng(n).random(n) < 0.1, full, 0).astype(np.int32)
        ref = oracle.color_d1(g, seed=2, init=init)
        got, st = gc.color_d1(dev(g.row_ptr), dev(g.col), init_colors=None if init is None else dev(init), **kw)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert st.rounds == ref.rounds and st.worklist == ref.worklist and st.num_colors == int(ref.colors.max())
    assert st.vertex_visits == ref.vertex_visits and st.edge_visits == ref.edge_visits
