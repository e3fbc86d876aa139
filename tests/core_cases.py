"""Graphs on which the largest tentative color falls while vertices that still
have to pass it are left: the vertices of high colors commit early, and their
neighbours climb past these colors later.  (On random graphs without initial
colors this hardly ever happens.)"""
import numpy as np

import graphgen as gg


def climb(path: int, top: int, low: int, star: int = 0):
    """A path, a clique of `top` vertices whose last one w takes color `top`,
    and a clique of `low` vertices, all adjacent to w and to the path's end:
    its vertices climb past color `top` only after w has committed it.  Keys
    fall from the far end of the path over the top clique to the low one.
    star: a separate star of so many leaves, which makes the library choose
    the incremental engine.  Returns (graph, explicit priorities)."""
    order = list(range(path + top + low))  # by key, highest first
    ps, ts, ls = order[:path], order[path:path + top], order[path + top:]
    e = [(ps[i], ps[i + 1]) for i in range(path - 1)]
    e += [(a, b) for i, a in enumerate(ts) for b in ts[i + 1:]]
    e += [(a, b) for i, a in enumerate(ls) for b in ls[i + 1:]]
    e += [(ts[-1], x) for x in ls]
    if path:
        e += [(ps[-1], x) for x in ls]
    n = len(order)
    if star:
        e += [(n, n + 1 + i) for i in range(star)]
        n += star + 1
    u, v = np.array(e).T
    prio = np.arange(n, 0, -1).astype(np.uint32) * 1000
    return gg.csr_from_pairs(n, u, v), prio


def climb_by_hash(path: int, top: int, low: int, star: int, seed: int):
    """climb with the ids laid out so that the default key gives that order."""
    import oracle
    g, _ = climb(path, top, low, star)
    by_key = np.argsort(-oracle.priorities(g.n, seed).astype(np.int64), kind="stable")
    m = path + top + low
    ids = np.empty(g.n, np.int64)
    core = np.sort(by_key[:m])  # the m ids of highest keys, in key order
    ids[:m] = by_key[:m]
    rest = np.setdiff1d(np.arange(g.n), core)
    ids[m:] = rest
    r = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    return gg.csr_from_pairs(g.n, ids[r], ids[g.col])


def anchored(m: int, p: float, share: float, steps: int, seed: int):
    """m uncolored vertices in G(m, p); about `share` of them are also joined
    to the committed vertices of colors 1 .. k_i, k_i up to steps, so that
    their colors start high.  Returns (graph, initial colors)."""
    rng = np.random.default_rng(seed)
    k = np.where(rng.random(m) < share, rng.integers(0, steps + 1, m), 0)
    i = np.repeat(np.arange(m), k)
    j = np.concatenate([np.arange(x) for x in k])
    u, v = np.nonzero(np.triu(rng.random((m, m)) < p, 1))
    g = gg.csr_from_pairs(m + steps, np.concatenate([i, u]), np.concatenate([j + m, v]))
    init = np.zeros(m + steps, np.int32)
    init[m:] = np.arange(1, steps + 1)
    return g, init


def five():
    """K4 on w, x, y, v (keys in this order) with colors 1..6 forbidden, and
    u, adjacent to v only, with 1..9 forbidden: v has to pass u's 10."""
    w, x, y, v, u = range(5)
    e = [(w, x), (w, y), (w, v), (x, y), (x, v), (y, v), (v, u)]
    e += [(a, 5 + c) for a in (w, x, y, v) for c in range(6)] + [(u, 5 + c) for c in range(9)]
    a, b = np.array(e).T
    init = np.zeros(14, np.int32)
    init[5:] = np.arange(1, 10)
    prio = np.arange(14, 0, -1).astype(np.uint32)
    return gg.csr_from_pairs(14, a, b), init, prio


def beside(g, prio, n: int, seed: int):
    """g and, separate from it, a random graph of n vertices: g's vertices
    reach the one-workgroup stage from an earlier one."""
    h = gg.erdos_renyi(n, 24.0, seed)
    row_ptr = np.concatenate([g.row_ptr, g.row_ptr[-1] + h.row_ptr[1:]]).astype(np.int32)
    col = np.concatenate([g.col, h.col + g.n]).astype(np.int32)
    rng = np.random.default_rng(seed)
    both = np.concatenate([prio, rng.integers(0, int(prio.max()), n)]).astype(np.uint32)
    return gg.Graph(g.n + n, row_ptr, col), both


CLIMBS = [(20, 4, 4), (20, 4, 7), (7, 4, 4), (1, 4, 4), (0, 4, 4), (60, 12, 15), (60, 30, 40), (60, 33, 40),
          (80, 40, 45), (40, 100, 20), (100, 70, 80)]
ANCHORED = [(8, 0.7, 24), (40, 0.5, 24), (150, 0.3, 24), (150, 0.5, 40), (300, 0.2, 24), (300, 0.4, 150),
            (700, 0.2, 60), (1000, 0.3, 150), (250, 0.8, 300), (120, 0.9, 700)]
