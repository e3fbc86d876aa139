"""Ghost steps from every kind of initial coloring (none, some vertices, all of
them: no ghost-blind phase) against the oracle, on local graphs whose entries
are dense in the rows and on ones whose rows are mostly empty (the boundary
detect's rows beyond its LDS table)."""
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


def graph(name):
    rng = np.random.default_rng(8)
    if name == "dense":
        return gg.rmat(13, 16, 4)
    # 3000 edges among 100000 vertices: 2048 entries of owned rows span far more than 2048 rows
    u, v = rng.integers(0, 100000, 3000), rng.integers(0, 100000, 3000)
    return gg.csr_from_pairs(100000, u, v, True)


@pytest.mark.parametrize("engine", [0, 1, 2])
@pytest.mark.parametrize("init", ["none", "some", "all"])
@pytest.mark.parametrize("name", ["dense", "empty rows"])
def test_steps(gc, name, init, engine):
    g = graph(name)
    lg = gg.ghost_local_graph(g, gg.hash_partition(g.n, 2, 5), 0, 1, np.random.default_rng(3).integers(1, 4, g.n))
    start = None
    if init != "none":
        start = oracle.color_d1_ghost(lg, seed=9).colors
        lg.ghost_colors = np.random.default_rng(4).integers(1, 4, lg.n_ghost).astype(np.int32)
        if init == "some":
            start = np.where(np.random.default_rng(5).random(lg.n_owned) < 0.3, 0, start).astype(np.int32)
    ref = oracle.color_d1_ghost(lg, seed=9, init_owned=start)
    got, rl, st = gc.color_d1_ghost_step(
        lg.n_owned, lg.n_ghost, 1, lg.n_g1, dev(lg.row_ptr), dev(lg.col), dev(lg.gid), dev(lg.ghost_colors), seed=9,
        init_owned=None if start is None else dev(start), trace_cap=4096, params=gc.Params(engine=engine))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert np.array_equal(rl.cpu().numpy()[:lg.n_ghost], ref.remote_loser)
    assert st.boundary_conflicts == ref.boundary_conflicts > 0 and st.remote_losers == ref.remote_losers
    assert st.rounds == ref.rounds and st.num_colors == ref.num_colors
