"""The work that a user of this library has it do, as measured cases: colorings
through the public entry points over the range of graph classes, sizes, kinds
(distance-1, distance-2, partial distance-2) and forms (one graph, one rank's
ghost step, several ranks, batched, served).

Graphs are made on the GPU from the seed alone: Erdos-Renyi graphs, 2D and 3D
stencil meshes, R-MAT graphs with (a, b, c) = (0.57, 0.19, 0.19), and patterns
whose column degrees follow a power law.  Every graph is symmetric CSR without
self-loops or duplicates; a pattern is given in CSR and CSC.
"""
import math

import numpy as np
import torch

import paper_2107_00075_amd as gc

DEV = "cuda"


def listed():
    return [
        # A small graph alone, as in a solver's setup phase or a request of its own: launches, host
        # round trips and the latency of each round are all there is.
        {"name": "d1_er_10k", "form": "d1", "graph": "er", "n": 10_000, "degree": 16},
        # A finite-element mesh with full 27-point coupling, colored for parallel assembly or
        # Gauss-Seidel sweeps: even degrees, few rounds.
        {"name": "d1_mesh27_128", "form": "d1", "graph": "mesh", "points": 27, "x": 128, "y": 128, "z": 128},
        # The largest single graph: a social-network-like graph with hubs of 10^5 neighbours and
        # hundreds of rounds, most of them small.
        {"name": "d1_rmat22", "form": "d1", "graph": "rmat", "scale": 22, "edge_factor": 16},
        # An ordinary skewed graph with the recolorDegrees key, the option that users take for fewer colors.
        {"name": "d1_rmat17_degrees", "form": "d1", "graph": "rmat", "scale": 17, "edge_factor": 16,
         "recolor_degrees": True},
        # Distance-2 coloring of a 7-point mesh, for compressed Jacobians and Hessians of PDE codes.
        {"name": "d2_mesh7_96", "form": "d2", "graph": "mesh", "points": 7, "x": 96, "y": 96, "z": 96},
        # Distance-2 coloring of an unstructured graph of an odd size: two-hop neighbourhoods of about
        # a thousand vertices and as many rounds as colors.
        {"name": "d2_er_20k", "form": "d2", "graph": "er", "n": 20_011, "degree": 32},
        # Partial distance-2 coloring of the columns of a large rectangular pattern with a few very
        # dense columns: sparse least-squares and Jacobian compression at full size.
        {"name": "pd2_4m_1m", "form": "pd2", "rows": 4_000_000, "cols": 1_000_000, "per_row": 8},
        # The same kind of pattern at an ordinary size.
        {"name": "pd2_200k_50k", "form": "pd2", "rows": 200_000, "cols": 50_000, "per_row": 8},
        # One rank's step of the distributed method: part 0 of 16 of a skewed graph, with one ghost
        # layer whose colors came from the neighbours.
        {"name": "ghost_rmat22_of16", "form": "ghost", "graph": "rmat", "scale": 22, "edge_factor": 16, "parts": 16},
        # The whole distributed method over 8 ranks on one GPU: many ghost steps from a partial
        # coloring, with few vertices left to recolor in each.
        {"name": "dist_rmat17_of8", "form": "dist", "graph": "rmat", "scale": 17, "edge_factor": 16, "parts": 8},
        # A batch of small and mid-size graphs of mixed kinds and classes in one call.
        {"name": "batch_48", "form": "batch", "jobs": 48, "n_max": 30_000},
        # The same kind of jobs served from host arrays: submitted, run together and read back.
        {"name": "serve_48", "form": "serve", "jobs": 48, "n_max": 30_000},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_mesh(rng, n_max, points):
    if points in (5, 9):
        side = _log_int(rng, 32, int(n_max ** 0.5))
        return {"graph": "mesh", "points": points, "x": side, "y": max(2, side - rng.randrange(8)), "z": 1}
    side = _log_int(rng, 10, int(n_max ** (1 / 3)))
    return {"graph": "mesh", "points": points, "x": side, "y": max(2, side - rng.randrange(4)),
            "z": max(2, side - rng.randrange(4))}


def draw(rng):
    form = rng.choice(["d1", "d1", "d1", "d2", "d2", "pd2", "pd2", "ghost", "dist", "batch", "serve"])
    if form == "d1":
        graph = rng.choice(["er", "mesh", "rmat"])
        if graph == "er":
            c = {"graph": "er", "n": _log_int(rng, 1_000, 2_000_000), "degree": rng.randint(8, 32)}
        elif graph == "mesh":
            c = _draw_mesh(rng, 2_097_152, rng.choice([5, 9, 7, 27]))
        else:
            c = {"graph": "rmat", "scale": rng.randint(10, 21), "edge_factor": rng.randint(8, 16)}
        if rng.random() < 0.25:
            c["recolor_degrees"] = True
        return {"form": "d1", **c}
    if form == "d2":
        if rng.random() < 0.5:
            return {"form": "d2", **_draw_mesh(rng, 884_736, rng.choice([5, 9, 7]))}
        return {"form": "d2", "graph": "er", "n": _log_int(rng, 1_000, 20_000), "degree": rng.randint(8, 32)}
    if form == "pd2":
        rows = _log_int(rng, 10_000, 2_000_000)
        return {"form": "pd2", "rows": rows, "cols": max(2_000, int(rows * rng.uniform(0.2, 0.5))),
                "per_row": rng.randint(4, 8)}
    if form == "ghost":
        return {"form": "ghost", "graph": "rmat", "scale": rng.randint(14, 21), "edge_factor": rng.randint(8, 16),
                "parts": rng.choice([4, 8, 16])}
    if form == "dist":
        return {"form": "dist", "graph": "rmat", "scale": rng.randint(12, 16), "edge_factor": rng.randint(8, 16),
                "parts": rng.randint(2, 8)}
    return {"form": form, "jobs": rng.randint(8, 48), "n_max": _log_int(rng, 2_000, 30_000)}


# ---------------------------------------------------------------------------
# graphs, on the GPU
# ---------------------------------------------------------------------------

def _csr(n, u, v):
    """Symmetric CSR of an edge list: self-loops and duplicates dropped, rows sorted."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    src = torch.div(key, n, rounding_mode="floor")
    return _row_ptr(src, n), (key - src * n).to(torch.int32)


def _row_ptr(sorted_rows, n):
    at = torch.arange(n + 1, device=DEV, dtype=sorted_rows.dtype)
    return torch.searchsorted(sorted_rows, at).to(torch.int32)


def _er(n, degree, gen):
    m = int(round(n * degree / 2))
    u = torch.randint(0, n, (m,), device=DEV, generator=gen)
    v = torch.randint(0, n, (m,), device=DEV, generator=gen)
    return _csr(n, u, v)


def _rmat(scale, edge_factor, gen):
    n, m = 1 << scale, edge_factor << scale
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for level in range(scale):
        r = torch.rand(m, device=DEV, generator=gen)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(n, device=DEV, generator=gen)
    return _csr(n, perm[u], perm[v])


def _mesh(x, y, z, points):
    ids = torch.arange(x * y * z, device=DEV)
    px, py, pz = ids % x, ids // x % y, ids // (x * y)
    star = points in (5, 7)
    cols = []
    for dz in ((0,) if points in (5, 9) else (-1, 0, 1)):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dx, dy, dz) == (0, 0, 0) or (star and abs(dx) + abs(dy) + abs(dz) > 1):
                    continue
                inside = ((px + dx >= 0) & (px + dx < x) & (py + dy >= 0) & (py + dy < y)
                          & (pz + dz >= 0) & (pz + dz < z))
                cols.append(torch.where(inside, ids + dx + x * (dy + y * dz), -1))
    cols = torch.stack(cols, 1)  # ascending within a row
    row_ptr = torch.zeros(x * y * z + 1, dtype=torch.int64, device=DEV)
    torch.cumsum((cols >= 0).sum(1), 0, out=row_ptr[1:])
    return row_ptr.to(torch.int32), cols[cols >= 0].to(torch.int32)


def _graph(case, gen):
    if case["graph"] == "er":
        return _er(case["n"], case["degree"], gen)
    if case["graph"] == "rmat":
        return _rmat(case["scale"], case["edge_factor"], gen)
    return _mesh(case["x"], case["y"], case["z"], case["points"])


def _pattern(rows, cols, per_row, gen):
    """rows x cols pattern with per_row distinct columns a row, column weights j^(-1/1.1): CSR and CSC."""
    cdf = np.cumsum(np.arange(1, cols + 1, dtype=np.float64) ** (-1 / 1.1))
    cdf = torch.from_numpy(cdf / cdf[-1]).to(DEV)

    def some(shape):
        r = torch.rand(shape, dtype=torch.float64, device=DEV, generator=gen)
        return torch.searchsorted(cdf, r).clamp_(max=cols - 1)

    c = some((rows, per_row))
    while True:
        c = c.sort(1).values
        again = torch.zeros_like(c, dtype=torch.bool)
        again[:, 1:] = c[:, 1:] == c[:, :-1]
        k = int(again.sum())
        if k == 0:
            break
        c[again] = some((k,))
    c = torch.randperm(cols, device=DEV, generator=gen)[c].sort(1).values
    row_ptr = torch.arange(0, rows * per_row + 1, per_row, dtype=torch.int32, device=DEV)
    r = torch.arange(rows, device=DEV)[:, None].expand(rows, per_row)
    key = (c * rows + r).reshape(-1).sort().values
    by_col = torch.div(key, rows, rounding_mode="floor")
    return (row_ptr, c.reshape(-1).to(torch.int32), _row_ptr(by_col, cols),
            (key - by_col * rows).to(torch.int32))


def _parts(row_ptr, col, parts, gen):
    """The local graph of every rank (owned vertices, then one ghost layer), the owners a random even split."""
    n = row_ptr.numel() - 1
    owner = torch.randperm(n, device=DEV, generator=gen) % parts
    index = torch.empty(n, dtype=torch.int64, device=DEV)
    owned = [torch.nonzero(owner == p).reshape(-1) for p in range(parts)]
    for o in owned:
        index[o] = torch.arange(o.numel(), device=DEV)
    src = torch.repeat_interleave(torch.arange(n, device=DEV), torch.diff(row_ptr).long())
    col = col.long()
    for p, o in enumerate(owned):
        mine = owner[src] == p
        s, c = index[src[mine]], col[mine]
        away = owner[c] != p
        ghosts = torch.unique(c[away])
        local = torch.where(away, o.numel() + torch.searchsorted(ghosts, c), index[c])
        order = torch.argsort(s * (o.numel() + ghosts.numel()) + local)
        yield {"n_owned": o.numel(), "n_ghost": ghosts.numel(), "layers": 1, "n_g1": ghosts.numel(),
               "row_ptr": _row_ptr(s, o.numel()), "col_idx": local[order].to(torch.int32),
               "gid": torch.cat([o, ghosts]).to(torch.int32), "ghost_owner": owner[ghosts].to(torch.int32),
               "ghost_index": index[ghosts].to(torch.int32)}


def _jobs(case, gen, seed):
    """Jobs of mixed kinds and classes: 70% D1, 20% D2, 10% PD2 on a graph's square pattern; sizes
    log-uniform; the power-law graphs among the D1 jobs.  The case fixes the mix, the seed the graphs."""
    rng = np.random.default_rng([case["jobs"], case["n_max"]])
    jobs = []
    for i in range(case["jobs"]):
        n = int(round(math.exp(rng.uniform(math.log(1_000), math.log(case["n_max"])))))
        kind = (gc.KIND_D1, gc.KIND_D2, gc.KIND_PD2)[int(np.searchsorted([0.7, 0.9], rng.random(), "right"))]
        family = rng.choice(["er", "mesh", "rmat"] if kind == gc.KIND_D1 else ["er", "mesh"])
        if family == "er":
            row_ptr, col = _er(n, int(rng.integers(8, 65)), gen)
        elif family == "rmat":
            row_ptr, col = _rmat(int(round(math.log2(n))), int(rng.integers(8, 17)), gen)
        else:
            points = int(rng.choice([5, 9, 7, 27]))
            flat = points in (5, 9)
            side = max(2, int(round(n ** (1 / 2 if flat else 1 / 3))))
            row_ptr, col = _mesh(side, side, 1 if flat else side, points)
        job = {"kind": kind, "row_ptr": row_ptr, "col_idx": col, "seed": (seed + i) & 0x7FFFFFFF}
        if kind == gc.KIND_PD2:  # symmetric: the CSC of the pattern is its CSR
            job.update(col_ptr=row_ptr, row_idx=col)
        jobs.append(job)
    return jobs


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    s = {"form": case["form"], "seed": (seed * 2654435761 + 1) & 0x7FFFFFFF}
    if case["form"] in ("d1", "d2"):
        s["graph"] = _graph(case, gen)
        s["params"] = gc.Params(flags=gc.COLOR_FLAG_RECOLOR_DEGREES) if case.get("recolor_degrees") else None
        s["out"] = torch.empty(s["graph"][0].numel() - 1, dtype=torch.int32, device=DEV)
    elif case["form"] == "pd2":
        s["graph"] = _pattern(case["rows"], case["cols"], case["per_row"], gen)
        s["out"] = torch.empty(case["cols"], dtype=torch.int32, device=DEV)
    elif case["form"] == "ghost":
        row_ptr, col = _graph(case, gen)
        most = int(torch.diff(row_ptr).max())
        s["part"] = p = next(_parts(row_ptr, col, case["parts"], gen))
        s["ghost_colors"] = torch.randint(1, most + 2, (p["n_ghost"],), dtype=torch.int32, device=DEV, generator=gen)
        s["out"] = torch.empty(p["n_owned"], dtype=torch.int32, device=DEV)
        s["ghosts"] = p["gid"][p["n_owned"]:].long()
        s["lost"] = torch.zeros(row_ptr.numel() - 1, dtype=torch.uint8, device=DEV)
    elif case["form"] == "dist":
        s["parts"] = list(_parts(*_graph(case, gen), case["parts"], gen))
        for p in s["parts"]:
            p["out"] = torch.empty(p["n_owned"], dtype=torch.int32, device=DEV)
    else:
        s["jobs"] = _jobs(case, gen, seed)
        if case["form"] == "batch":  # one result buffer, a slice of it for each job
            sizes = [j["row_ptr"].numel() - 1 for j in s["jobs"]]
            s["out"] = torch.empty(sum(sizes), dtype=torch.int32, device=DEV)
            for j, o in zip(s["jobs"], torch.split(s["out"], sizes)):
                j["out"] = o
        else:
            names = ("row_ptr", "col_idx", "col_ptr", "row_idx")
            s["jobs"] = [(j["kind"], [j[k].cpu().numpy() if k in j else None for k in names], j["seed"])
                         for j in s["jobs"]]
            s["server"] = gc.ColorServer(1 << 31, 64)
    return s


def run(s):
    form = s["form"]
    if form == "d1":
        colors, st = gc.color_d1(*s["graph"], seed=s["seed"], out=s["out"], params=s["params"])
        return colors, st.rounds, st.num_colors
    if form == "d2":
        colors, st = gc.color_d2(*s["graph"], seed=s["seed"], out=s["out"], params=s["params"])
        return colors, st.rounds, st.num_colors
    if form == "pd2":
        colors, st = gc.color_pd2(*s["graph"], seed=s["seed"], out=s["out"])
        return colors, st.rounds, st.num_colors
    if form == "ghost":
        p = s["part"]
        colors, lost, st = gc.color_d1_ghost(p["n_owned"], p["n_ghost"], 1, p["n_g1"], p["row_ptr"], p["col_idx"],
                                             p["gid"], s["ghost_colors"], seed=s["seed"], out=s["out"])
        s["lost"].index_copy_(0, s["ghosts"], lost)  # by global id, as the owners are told
        return colors, s["lost"], st.boundary_conflicts, st.rounds, st.num_colors
    if form == "dist":
        colors, st = gc.color_d1_distributed(s["parts"], seed=s["seed"])
        return colors, st.detects, st.num_colors, st.exchanged_total
    if form == "batch":
        gc.color_batch(s["jobs"])
        return s["out"]
    server = s["server"]
    ids = [server.submit(kind, *arrays, seed=seed)[0] for kind, arrays, seed in s["jobs"]]
    server.drain()
    return [server.poll(i)[0] for i in ids]


def _sizes(case):
    """(vertices, adjacency entries) of a case's graph; for R-MAT the entries that are left of
    2 * edge_factor * n once duplicates are dropped, about."""
    if case["graph"] == "er":
        return case["n"], case["n"] * case["degree"]
    if case["graph"] == "rmat":
        n = 1 << case["scale"]
        return n, int(2 * case["edge_factor"] * n * (1 - 0.19 * 0.84 ** (case["scale"] - 14)))
    x, y, z = case["x"], case["y"], case["z"]
    if case["points"] in (5, 7):
        nnz = 2 * ((x - 1) * y * z + x * (y - 1) * z + x * y * (z - 1))
    else:
        nnz = (3 * x - 2) * (3 * y - 2) * (3 * z - 2 if z > 1 else 1) - x * y * z
    return x * y * z, nnz


def work(case):
    """Every graph array read once, every color written once; the path has no floating-point operations."""
    form = case["form"]
    if form == "pd2":
        nnz = case["rows"] * case["per_row"]
        total = 4 * (case["rows"] + 2 * case["cols"] + 2 * nnz)
    elif form in ("batch", "serve"):
        # n log-uniform in [1000, n_max]: mean (n_max - 1000) / log(n_max / 1000); about 22 entries a vertex
        n = (case["n_max"] - 1_000) / math.log(case["n_max"] / 1_000)
        total = case["jobs"] * n * 4 * (2 + 22)
    else:
        n, nnz = _sizes(case)
        if form == "ghost":
            n, nnz = n / case["parts"], nnz / case["parts"]
            total = 4 * (2 * n + nnz) + 13 * min(nnz, n * case["parts"])  # a ghost's id, color and flag
        elif form == "dist":
            total = 4 * (2 * n + nnz) + 16 * min(nnz, n * case["parts"])  # a ghost's id, owner, index and color
        else:
            total = 4 * (2 * n + nnz)
    return {"bytes": float(total), "flops": 0.0}


# ---------------------------------------------------------------------------
# the same colorings by sorting, in 64-bit integers
# ---------------------------------------------------------------------------

def _mix(h):
    m = 0xFFFFFFFF
    h = h ^ (h >> 16)
    h = h * 0x85EBCA6B & m
    h = h ^ (h >> 13)
    h = h * 0xC2B2AE35 & m
    return h ^ (h >> 16)


def _rounds(n, src, dst, key):
    """Synchronous first-fit rounds over the directed pairs (src, dst): each uncolored vertex tries the
    smallest color that no colored neighbour has, and keeps it unless an uncolored neighbour of higher
    key tries the same."""
    colors = torch.zeros(n, dtype=torch.int64, device=DEV)
    rounds = 0
    while bool((colors == 0).any()):
        rounds += 1
        live = colors[src] == 0
        src, dst = src[live], dst[live]
        c = colors[dst]
        pairs = torch.unique((src * (n + 1) + c)[c > 0])
        owner = torch.div(pairs, n + 1, rounding_mode="floor")
        first = torch.searchsorted(owner, owner)
        in_a_row = pairs - owner * (n + 1) == torch.arange(pairs.numel(), device=DEV) - first + 1
        tried = 1 + torch.bincount(owner[in_a_row], minlength=n)
        beaten = (c == 0) & (tried[dst] == tried[src]) & (key[dst] > key[src])
        wins = colors == 0
        wins[src[beaten]] = False
        colors[wins] = tried[wins]
    return colors, rounds, int(colors.max()) if n else 0


def exact(case, seed):
    if case["form"] not in ("d1", "d2", "pd2") or case.get("graph") == "rmat" or case.get("recolor_degrees"):
        return None
    if case["form"] == "pd2" or (case["form"] == "d2" and case["graph"] == "er" and case["n"] * case["degree"] > 60_000):
        return None
    s = prepare(case, seed)
    row_ptr, col = (t.long() for t in s["graph"])
    n, deg = row_ptr.numel() - 1, torch.diff(row_ptr)
    src = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    if case["form"] == "d2":
        d2 = deg[col]
        start = torch.repeat_interleave(row_ptr[:-1][col] - (torch.cumsum(d2, 0) - d2), d2)
        far = col[start + torch.arange(start.numel(), device=DEV)]
        src2 = torch.repeat_interleave(src, d2)
        keep = far != src2
        src, col = torch.cat([src, src2[keep]]), torch.cat([col, far[keep]])
    ids = torch.arange(n, device=DEV)
    key = _mix(ids ^ _mix((s["seed"] ^ 0x9E3779B9) & 0xFFFFFFFF))
    return _rounds(n, src, col, key)
