"""Two-hop list building against the oracle: first hops at the edges of the
groups that walk them, rows of very different lengths, lists at the length
from which duplicates are removed, and heavy columns of one and several units
with id ranges at the edges of the bitmaps held in LDS."""
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


def pattern(n_rows, n_cols, rows, cols):
    """The pattern of the entries (rows[i], cols[i]), repeated entries once."""
    key = np.unique(np.asarray(rows, np.int64) * n_cols + np.asarray(cols, np.int64))
    r, c = key // n_cols, key % n_cols
    by_col = np.lexsort((r, c))
    ptr = lambda ids, n: np.concatenate(([0], np.cumsum(np.bincount(ids, minlength=n)))).astype(np.int32)
    return gg.Bipartite(n_rows, n_cols, ptr(r, n_rows), c.astype(np.int32), ptr(c, n_cols),
                        r[by_col].astype(np.int32))


def check_pd2(gc, b, seed):
    ref = oracle.color_pd2(b, seed=seed)
    got, st = gc.color_pd2(dev(b.row_ptr), dev(b.col_idx), dev(b.col_ptr), dev(b.row_idx), seed=seed, trace_cap=4096,
                           params=gc.Params(engine=gc.ENGINE_INCREMENTAL))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert st.rounds == ref.rounds and st.worklist == ref.worklist
    assert st.vertex_visits == ref.vertex_visits and st.edge_visits == ref.edge_visits


# groups of 16 lanes to 16 entries, a wavefront to 1024, a unit to 32768
# entries of a heavy column; rows of 1 to several hundred entries
@pytest.mark.parametrize("hop", [1, 15, 16, 17, 63, 64, 65, 129, 1023, 1024, 1025, 4097])
def test_first_hops(gc, hop):
    rng = np.random.default_rng(hop)
    n_rows, n_cols = 6000, 3000
    cols = rng.choice(n_cols, 3, replace=False)
    rows = np.concatenate([rng.choice(n_rows, hop, replace=False) for _ in cols])
    others = np.setdiff1d(np.arange(n_cols), cols)
    wide = rng.integers(0, n_rows, 4)
    b = pattern(n_rows, n_cols,
                np.concatenate((rows, rng.integers(0, n_rows, 6000), np.repeat(wide, [3, 60, 200, 500]))),
                np.concatenate((np.repeat(cols, hop), rng.choice(others, 6763))))
    check_pd2(gc, b, 2)


# one column of `hop` rows with k others each, all from a pool of 40: the
# list has hop * k entries of at most 40 distinct ones
@pytest.mark.parametrize("hop, k", [(1024, 4), (241, 17), (1024, 39)])
def test_list_duplicates(gc, hop, k):
    rng = np.random.default_rng(k)
    rows = np.repeat(np.arange(hop), k + 1)
    cols = np.concatenate([np.concatenate(([0], 1 + rng.choice(40, k, replace=False))) for _ in range(hop)])
    check_pd2(gc, pattern(hop, 41, rows, cols), 3)


# bitmaps of n / 32 + 1 words: in LDS to 4096 words by several workgroups a
# CU, to 37376 by one, in memory above; a column of one unit, one of two, and
# lists with duplicates that are made sets by the same bitmaps
@pytest.mark.parametrize("n_cols", [131071, 131072, 1196031, 1196032])
@pytest.mark.parametrize("hop", [32768, 32769])
def test_heavy_columns_and_id_range(gc, n_cols, hop):
    rng = np.random.default_rng(hop)
    n_rows = 40000
    rows = [rng.choice(n_rows, h, replace=False) for h in (hop, 1025, 700)]
    cols = [np.full(len(r), c) for r, c in zip(rows, (n_cols - 1, 0, 77))]
    more = rng.integers(0, n_cols, 2 * n_rows)
    pool = rng.integers(0, n_cols, 50)
    few = rng.choice(rows[2], 9 * 700)
    b = pattern(n_rows, n_cols, np.concatenate((*rows, np.repeat(np.arange(n_rows), 2), few)),
                np.concatenate((*cols, more, rng.choice(pool, len(few)))))
    check_pd2(gc, b, 4)


# hubs adjacent to each other and to tens of thousands of vertices: they lose
# for many rounds with lists on both sides of the length that is compacted a
# window at a time, in the per-round kernels and in the tail kernel
@pytest.mark.parametrize("flags, tail", [("COLOR_FLAG_NO_TAIL", 0), (None, 1 << 30), (None, 0)])
@pytest.mark.parametrize("leaves", [16000, 17000, 50000])
def test_long_lists(gc, leaves, flags, tail):
    rng = np.random.default_rng(leaves)
    n, hubs = 80000, 24
    u = np.concatenate((np.repeat(np.arange(hubs), leaves), np.repeat(np.arange(hubs), hubs), rng.integers(0, n, 200000)))
    v = np.concatenate([rng.choice(n, leaves, replace=False) for _ in range(hubs)]
                       + [np.tile(np.arange(hubs), hubs), rng.integers(0, n, 200000)])
    perm = rng.permutation(n)
    g = gg.csr_from_pairs(n, perm[u], perm[v], True)
    ref = oracle.color_d1(g, seed=6)
    got, st = gc.color_d1(dev(g.row_ptr), dev(g.col), seed=6, trace_cap=4096,
                          params=gc.Params(engine=gc.ENGINE_INCREMENTAL, tail_threshold=tail,
                                           flags=getattr(gc, flags) if flags else 0))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref.colors)
    assert st.rounds == ref.rounds > 10 and st.worklist == ref.worklist
    assert st.vertex_visits == ref.vertex_visits and st.edge_visits == ref.edge_visits
