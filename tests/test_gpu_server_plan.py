"""The arena space the server plans for a job with long two-hop walks: what the
engine uses, and no more."""
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


def up(x):
    return (x + 255) // 256 * 256


def planned_bytes(n, nnz, entries, words_per_vertex):
    """The job's arrays and the incremental engine's buffers, without the
    bitmaps of the duplicate removal (in LDS for ids below 1196032) and without
    the scan's storage."""
    b = up(4 * (n + 1)) + up(4 * nnz) + up(4 * n)
    b += 2048 + 6 * up(4 * n) + up(n) + 256 + up(8 * n) + 6 * up(4 * (n + 1))
    b += up(4 * words_per_vertex * n) + 2 * up(4 * entries) + 256 + 2 * up(16 * n) + up((n + 3) // 4 * 4)
    return b + up(4 * (n // 32 + 1))


def test_no_space_for_bitmaps_that_are_in_lds(gc):
    n = 100_000
    i = np.arange(n)
    g = gg.csr_from_pairs(n, np.tile(i, 6), np.concatenate([(i + k) % n for k in range(1, 7)]))
    # degree 12: 12 * 13 - 12 = 144 entries per list, five bitset words; the bitmaps would be 3.2 MB
    budget = planned_bytes(n, g.nnz, 144 * n, 144 // 32 + 1) + 1_500_000
    srv = gc.ColorServer(budget, max_slots=2)
    try:
        jid, _ = srv.submit(2, g.row_ptr, g.col, seed=3)
        srv.drain()
        colors, st = srv.poll(jid)
    finally:
        srv.close()
    assert st.engine == gc.ENGINE_INCREMENTAL
    assert np.array_equal(colors, oracle.color_d2(g, seed=3).colors)
