"""Measured work: searches as a program that uses this library makes them.

A case is a dict of plain values.  ``kind`` names the entry point:

  single   bfs_run, one root on a resident graph
  noalloc  bfs_run_noalloc, one root on a plain CSR without a handle
  batch    bfs_run_batch, up to 64 roots in one call
  blocked  bfs_grid2d_run, the R x C grid of virtual processors
  serve    bfs_submit / bfs_server_completed / bfs_poll on a pool of graphs

``prepare`` builds the graph on the GPU from the seed (R-MAT with the usual
quadrant probabilities, ids relabelled at random, mirrored, loops and
duplicates dropped; or a 4-neighbour grid), creates the handle a program
keeps, picks roots of non-zero degree and allocates the result buffers.

The searches fill a parent array wherever a case says so, but parents are
not among the outputs: any neighbour one level nearer the root is a valid
parent, and which one a search stores depends on the order its threads run
in.  Levels and the search's own counts are unique and come back whole.
"""
import math

import torch

import paper_1408_1605_amd as bfsmi

A, B, C = 0.57, 0.19, 0.19  # R-MAT quadrant probabilities (D = 1 - A - B - C)
CHUNK = 1 << 26             # edges generated together
PART = 1 << 28              # mirrored edges sorted together


def listed():
    return [
        # the smallest calls: a plain CSR without a handle, where the call's
        # launches and waits are all there is
        {"name": "noalloc_rmat12", "kind": "noalloc", "graph": "rmat", "vertices": 1 << 12,
         "edgefactor": 16, "parents": True},
        # a small square mesh on a plain handle: a few hundred narrow levels
        {"name": "single_grid256", "kind": "single", "graph": "grid", "width": 256, "height": 256,
         "order": False, "direction": False, "parents": True},
        # a small social-network graph, levels and parents
        {"name": "single_rmat16", "kind": "single", "graph": "rmat", "vertices": 1 << 16,
         "edgefactor": 16, "order": True, "direction": False, "parents": True},
        # a vertex count that is no power of two, on the caller's own order,
        # levels only
        {"name": "single_ragged_plain", "kind": "single", "graph": "rmat", "vertices": 777777,
         "edgefactor": 9, "order": False, "direction": False, "parents": False},
        # the middle of the range: one-root-at-a-time at scale 22
        {"name": "single_rmat22", "kind": "single", "graph": "rmat", "vertices": 1 << 22,
         "edgefactor": 16, "order": True, "direction": False, "parents": True},
        # the headline workload
        {"name": "single_rmat26", "kind": "single", "graph": "rmat", "vertices": 1 << 26,
         "edgefactor": 16, "order": True, "direction": False, "parents": True},
        # the large-diameter graph: thousands of levels in one search
        {"name": "single_grid4096", "kind": "single", "graph": "grid", "width": 4096,
         "height": 4096, "order": True, "direction": False, "parents": True},
        # the direction-optimizing option on a large graph
        {"name": "direction_rmat24", "kind": "single", "graph": "rmat", "vertices": 1 << 24,
         "edgefactor": 16, "order": True, "direction": True, "parents": True},
        # a full batch of roots
        {"name": "batch64_rmat22", "kind": "batch", "graph": "rmat", "vertices": 1 << 22,
         "edgefactor": 16, "order": True, "roots": 64},
        # a few roots on a small plain graph of ragged size
        {"name": "batch5_ragged_plain", "kind": "batch", "graph": "rmat", "vertices": 50021,
         "edgefactor": 12, "order": False, "roots": 5},
        # the paper's 2D decomposition inside one GPU
        {"name": "blocked2x4_rmat20", "kind": "blocked", "graph": "rmat", "vertices": 1 << 20,
         "edgefactor": 16, "rows": 2, "columns": 4, "parents": True},
        # a burst of queries over graphs of several sizes, results delivered
        # into device buffers
        {"name": "serve_pool8", "kind": "serve", "rmat_graphs": 6, "rmat_low": 1 << 14,
         "rmat_high": 1 << 20, "edgefactor": 16, "grids": 2, "grid_low": 256, "grid_high": 512,
         "queries": 48},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "single", "noalloc", "batch", "batch",
                       "blocked", "serve"])
    if kind == "serve":
        low = _log_int(rng, 1 << 11, 1 << 15)
        side = _log_int(rng, 64, 300)
        return {"kind": "serve", "rmat_graphs": rng.randint(1, 6), "rmat_low": low,
                "rmat_high": _log_int(rng, 1 << 16, 1 << 20), "edgefactor": rng.randint(8, 16),
                "grids": rng.randint(0, 2), "grid_low": side, "grid_high": side + rng.randint(0, 212),
                "queries": rng.randint(4, 48)}
    if kind == "noalloc":
        if rng.random() < 0.5:
            return {"kind": kind, "graph": "rmat", "vertices": _log_int(rng, 1 << 8, 1 << 18),
                    "edgefactor": rng.randint(4, 16), "parents": rng.random() < 0.7}
        return {"kind": kind, "graph": "grid", "width": _log_int(rng, 4, 512),
                "height": _log_int(rng, 4, 512), "parents": rng.random() < 0.7}
    if kind == "batch":
        return {"kind": kind, "graph": "rmat", "vertices": _log_int(rng, 1 << 12, 1 << 22),
                "edgefactor": rng.randint(4, 16), "order": rng.random() < 0.7,
                "roots": rng.randint(1, 64)}
    if kind == "blocked":
        rows, columns = rng.choice([(1, 1), (2, 1), (2, 2), (8, 1), (1, 8), (2, 4), (4, 4)])
        return {"kind": kind, "graph": "rmat", "vertices": _log_int(rng, 1 << 14, 1 << 22),
                "edgefactor": rng.randint(8, 16), "rows": rows, "columns": columns,
                "parents": rng.random() < 0.7}
    if rng.random() < 0.3:
        return {"kind": kind, "graph": "grid", "width": _log_int(rng, 8, 3000),
                "height": _log_int(rng, 8, 3000), "order": rng.random() < 0.5, "direction": False,
                "parents": rng.random() < 0.7}
    return {"kind": kind, "graph": "rmat", "vertices": _log_int(rng, 1 << 12, 1 << 25),
            "edgefactor": rng.randint(4, 16), "order": rng.random() < 0.7,
            "direction": rng.random() < 0.25, "parents": rng.random() < 0.7}


# ---- inputs -----------------------------------------------------------------


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rmat_edges(n, scale, vertices, perm, gen):
    """n generated edges as relabelled endpoints, self-loops dropped."""
    u = torch.zeros(n, dtype=torch.int64, device="cuda")
    v = torch.zeros(n, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = torch.rand(n, generator=gen, device="cuda")
        down = r >= A + B
        right = ((r >= A) & ~down) | (r >= A + B + C)
        u.mul_(2).add_(down)
        v.mul_(2).add_(right)
    # any vertex count: scale the 2^scale ids down to it
    u = perm[u.mul_(vertices) >> scale]
    v = perm[v.mul_(vertices) >> scale]
    keep = u != v
    return u[keep], v[keep]


def _rmat(vertices, edgefactor, gen):
    """(row offsets int64, columns int32) of a symmetric R-MAT graph."""
    scale = max(1, (vertices - 1).bit_length())
    total = vertices * edgefactor
    parts = -(-2 * total // PART)
    step = -(-vertices // parts)
    perm = torch.randperm(vertices, generator=gen, device="cuda")
    held = [[] for _ in range(parts)]
    for at in range(0, total, CHUNK):
        u, v = _rmat_edges(min(CHUNK, total - at), scale, vertices, perm, gen)
        key = torch.cat([(u << 32) | v, (v << 32) | u])
        del u, v
        for p in range(parts):
            if parts == 1:
                held[p].append(key)
            else:
                row = key >> 32
                held[p].append(key[(row >= p * step) & (row < (p + 1) * step)])
    del perm
    off = torch.empty(vertices + 1, dtype=torch.int64, device="cuda")
    cols, before = [], 0
    for p in range(parts):
        key = torch.unique(torch.cat(held[p]))  # sorted by row, then column
        held[p] = None
        lo, hi = p * step, min(vertices, (p + 1) * step)
        rows = torch.arange(lo, hi + 1, dtype=torch.int64, device="cuda") << 32
        off[lo:hi + 1] = torch.searchsorted(key, rows) + before
        cols.append((key & 0xffffffff).to(torch.int32))
        before += key.numel()
        del key
    return off, (cols[0] if parts == 1 else torch.cat(cols))


def _grid(width, height):
    """4-neighbour grid, id = row * width + column, rows in ascending order."""
    ids = torch.arange(width * height, dtype=torch.int32, device="cuda")
    x, y = ids % width, torch.div(ids, width, rounding_mode="floor")
    near = torch.stack([ids - width, ids - 1, ids + 1, ids + width], dim=1)
    there = torch.stack([y > 0, x > 0, x < width - 1, y < height - 1], dim=1)
    off = torch.zeros(width * height + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(there.sum(dim=1), dim=0, out=off[1:])
    return off, near[there]


def _csr(case, gen):
    if case["graph"] == "grid":
        off, col = _grid(case["width"], case["height"])
    else:
        off, col = _rmat(case["vertices"], case["edgefactor"], gen)
    return off, col


def _roots(off, n, gen):
    """n distinct vertices of non-zero degree, uniform."""
    vertices = off.numel() - 1
    got = []
    while len(got) < n:
        tries = torch.randint(vertices, (4096,), generator=gen, device="cuda")
        for r in tries[off[tries + 1] > off[tries]].tolist():
            if r not in got and len(got) < n:
                got.append(r)
    return got


def _handle(off, col, flags):
    vertices, nnz = off.numel() - 1, col.numel()
    need = bfsmi.bfs_workspace_bytes(vertices, nnz, flags)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    handle = bfsmi.bfs_graph_create(vertices, nnz, off, col, ws, need, flags)
    return bfsmi.Graph(vertices, nnz, off, col, ws, handle)


class _Pool:
    """A server over resident graphs; closes the server before the graphs."""

    def __init__(self, graphs, arena_bytes):
        self.graphs = graphs
        self.arena = torch.empty(arena_bytes, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        self.server = bfsmi.bfs_server_create(self.arena, max_lanes=64, max_inflight=len(graphs))
        self.ids = [bfsmi.bfs_server_add_graph(self.server, g.handle) for g in graphs]

    def __del__(self):
        if getattr(self, "server", None):
            bfsmi.bfs_server_destroy(self.server)
            self.server = 0


def _spread(low, high, n):
    """n sizes from low to high, equal ratios apart."""
    if n == 1:
        return [high]
    return [int(round(low * (high / low) ** (i / (n - 1)))) for i in range(n)]


def _pool_csrs(case, gen):
    for v in _spread(case["rmat_low"], case["rmat_high"], case["rmat_graphs"]):
        yield _rmat(v, case["edgefactor"], gen), None
    if case["grids"]:
        for s in _spread(case["grid_low"], case["grid_high"], case["grids"]):
            yield _grid(s, s), s


def _queries(case, csrs, seed):
    """(graph, root) of each query: graphs in turn, roots at random."""
    gen = _generator(seed + (1 << 40))
    roots = [_roots(off, -(-case["queries"] // len(csrs)), gen) for off, _ in csrs]
    return [(q % len(csrs), roots[q % len(csrs)][q // len(csrs)]) for q in range(case["queries"])]


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind == "serve":
        csrs = [c for c, _ in _pool_csrs(case, gen)]
        graphs = [_handle(off, col, bfsmi.BFS_DEGREE_ORDER) for off, col in csrs]
        queries = _queries(case, csrs, seed)
        out = [torch.empty(graphs[g].V, dtype=torch.int32, device="cuda") for g, _ in queries]
        return {"case": case, "pool": _Pool(graphs, 2 << 30), "queries": queries, "out": out}
    off, col = _csr(case, gen)
    vertices, nnz = off.numel() - 1, col.numel()
    state = {"case": case, "roots": _roots(off, case.get("roots", 1), gen)}
    if kind == "batch":
        flags = bfsmi.BFS_WS_BATCH | (bfsmi.BFS_DEGREE_ORDER if case["order"] else 0)
        state["graph"] = _handle(off, col, flags)
        state["levels"] = torch.empty((case["roots"], vertices), dtype=torch.int8, device="cuda")
        return state
    state["levels"] = torch.empty(vertices, dtype=torch.int32, device="cuda")
    state["parents"] = torch.empty_like(state["levels"]) if case["parents"] else None
    if kind == "noalloc":
        state["csr"] = (vertices, nnz, off, col)
    elif kind == "blocked":
        need = bfsmi.bfs_grid2d_workspace_bytes(vertices, nnz, case["rows"], case["columns"])
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        handle = bfsmi.bfs_grid2d_create(vertices, nnz, off, col, case["rows"], case["columns"], ws,
                                         need)
        state["graph"] = bfsmi.Grid2D(vertices, nnz, case["rows"], case["columns"], ws, handle)
    else:
        g = _handle(off, col, bfsmi.BFS_DEGREE_ORDER if case["order"] else 0)
        if case["direction"]:
            g.set_option(bfsmi.BFS_OPT_DIRECTION, 1)
        state["graph"] = g
    return state


# ---- one pass ---------------------------------------------------------------


def _answer(levels, st):
    return {"levels": levels, "depth": int(st.levels), "reached": int(st.reached),
            "edges": int(st.edges_scanned)}


def run(state):
    kind = state["case"]["kind"]
    if kind == "serve":
        pool, out = state["pool"], state["out"]
        waiting = {}
        for q, (g, root) in enumerate(state["queries"]):
            waiting[bfsmi.bfs_submit(pool.server, pool.ids[g], root)] = q
        while waiting:
            for t in bfsmi.bfs_server_completed(pool.server):
                bfsmi.bfs_poll(pool.server, t, out[waiting.pop(t)])
        return out
    if kind == "batch":
        st = bfsmi.bfs_run_batch(state["graph"].handle, state["roots"], state["levels"])
        return _answer(state["levels"], st)
    root, levels, parents = state["roots"][0], state["levels"], state["parents"]
    if kind == "noalloc":
        vertices, nnz, off, col = state["csr"]
        st = bfsmi.bfs_run_noalloc(vertices, nnz, off, col, root, levels, parents)
    elif kind == "blocked":
        st = bfsmi.bfs_grid2d_run(state["graph"].handle, root, levels, parents)
    else:
        st = bfsmi.bfs_run(state["graph"].handle, root, levels, parents)
    return _answer(levels, st)


# ---- what a pass cannot do without -------------------------------------------


def _size(case):
    """(vertices, CSR entries); R-MAT entries before duplicates merge."""
    if case["graph"] == "grid":
        w, h = case["width"], case["height"]
        return w * h, 2 * (2 * w * h - w - h)
    return case["vertices"], 2 * case["edgefactor"] * case["vertices"]


def work(case):
    """The CSR read once and the results written once; a bottom-up search
    reads one neighbour per vertex instead of all."""
    kind = case["kind"]
    if kind == "serve":
        sizes = [(v, 2 * case["edgefactor"] * v)
                 for v in _spread(case["rmat_low"], case["rmat_high"], case["rmat_graphs"])]
        if case["grids"]:
            sizes += [(s * s, 4 * s * s)
                      for s in _spread(case["grid_low"], case["grid_high"], case["grids"])]
        each = [case["queries"] // len(sizes) + (i < case["queries"] % len(sizes))
                for i in range(len(sizes))]
        return {"bytes": sum((8 * v + 4 * e if n else 0) + 4 * v * n
                             for (v, e), n in zip(sizes, each)), "flops": 0}
    v, e = _size(case)
    if kind == "batch":
        return {"bytes": 8 * v + 4 * e + v * case["roots"], "flops": 0}
    out = 8 * v if case["parents"] else 4 * v
    return {"bytes": 8 * v + 4 * (v if case.get("direction") else e) + out, "flops": 0}


# ---- the same results without the library --------------------------------------


def _hop_levels(off, col, root):
    """Hop distances from root, frontier by frontier; -1 where unreached."""
    vertices = off.numel() - 1
    levels = torch.full((vertices,), -1, dtype=torch.int64, device="cuda")
    levels[root] = 0
    front = torch.tensor([root], device="cuda")
    depth, edges = 0, 0
    while front.numel():
        depth += 1
        first, degree = off[front], off[front + 1] - off[front]
        upto = torch.cumsum(degree, 0)
        count = int(upto[-1])
        edges += count
        mark = torch.zeros(vertices, dtype=torch.bool, device="cuda")
        for lo in range(0, count, PART):  # edges lo .. hi of the frontier
            hi = min(count, lo + PART)
            e = torch.arange(lo, hi, dtype=torch.int64, device="cuda")
            k = torch.searchsorted(upto, e, right=True)
            mark[col[first[k] + e - (upto[k] - degree[k])].long()] = True
            del e, k
        front = torch.nonzero(mark & (levels < 0)).flatten()
        levels[front] = depth
    return levels, depth, edges


def _grid_levels(width, height, root):
    ids = torch.arange(width * height, device="cuda")
    x, y = ids % width, torch.div(ids, width, rounding_mode="floor")
    levels = (x - root % width).abs() + (y - root // width).abs()
    return levels, int(levels.max()) + 1, 2 * (2 * width * height - width - height)


def exact(case, seed):
    gen = _generator(seed)
    if case["kind"] == "serve":
        pool = list(_pool_csrs(case, gen))
        csrs = [c for c, _ in pool]
        return [(_hop_levels(*csrs[g], root) if pool[g][1] is None else
                 _grid_levels(pool[g][1], pool[g][1], root))[0]
                for g, root in _queries(case, csrs, seed)]
    off, col = _csr(case, gen)
    roots = _roots(off, case.get("roots", 1), gen)
    if case["graph"] == "grid":
        levels, depth, edges = _grid_levels(case["width"], case["height"], roots[0])
    elif case["kind"] == "batch":
        levels = torch.stack([_hop_levels(off, col, r)[0] for r in roots])
        # the union search's counts: a vertex enters the union frontier once
        # per level at which some root finds it
        degree = off[1:] - off[:-1]
        depth, edges, reached = int(levels.max()) + 1, 0, 0
        for d in range(depth):
            front = (levels == d).any(dim=0)
            reached += int(front.sum())
            edges += int(degree[front].sum())
        return {"levels": levels, "depth": depth, "reached": reached, "edges": edges}
    else:
        levels, depth, edges = _hop_levels(off, col, roots[0])
    return {"levels": levels, "depth": depth, "reached": int((levels >= 0).sum()), "edges": edges}
