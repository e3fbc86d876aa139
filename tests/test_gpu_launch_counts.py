"""Launch counts of a call: the pull engine's first round from no colors has no
color launch."""
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


@pytest.mark.parametrize("kind", ["d1", "d2", "pd2"])
@pytest.mark.parametrize("start", ["no colors", "some"])
def test_first_round_has_no_color_launch(gc, kind, start):
    g = gg.erdos_renyi(3000, 8, 1)
    init = None
    if start == "some":
        full = getattr(oracle, f"color_{kind if kind != 'pd2' else 'd2'}")(g, seed=7).colors
        init = np.where(np.arange(g.n) % 9 == 0, full, 0).astype(np.int32)
    kw = dict(seed=2, init_colors=None if init is None else dev(init),
              params=gc.Params(engine=gc.ENGINE_PULL, flags=gc.COLOR_FLAG_KERNEL_TIMING))
    if kind == "pd2":
        b = gg.square_pattern_bipartite(g)
        _, st = gc.color_pd2(dev(b.row_ptr), dev(b.col_idx), dev(b.col_ptr), dev(b.row_idx), **kw)
    else:
        _, st = getattr(gc, f"color_{kind}")(dev(g.row_ptr), dev(g.col), **kw)
    torch.cuda.synchronize()
    assert st.detect_launches - st.color_launches == (1 if init is None else 0)
    assert st.detect_launches >= st.rounds
