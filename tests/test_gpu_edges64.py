"""A graph of more than 2^32 edges through every search that holds a graph of
that size: vertices v and v + d mod 2^26 are neighbours for 67 differences d
(powers of two and three times powers of two, both signs).  The expected
levels come from the same differences, as shifts of whole arrays."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

V = 1 << 26
ROOT = V - 3
DIFFS = sorted({x % V for k in range(26) for x in (1 << k, -(1 << k))} |
               {x % V for k in range(8) for x in (3 << k, -(3 << k))})


@pytest.fixture(scope="module")
def graph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1408_1605_amd as p
    p.load()
    K = len(DIFFS)
    assert K * V > 1 << 32
    off = torch.arange(V + 1, device="cuda") * K
    col = torch.empty(K * V, dtype=torch.int32, device="cuda")
    ids = torch.arange(V, dtype=torch.int32, device="cuda")
    for k, d in enumerate(DIFFS):
        col.view(V, K)[:, k] = (ids + d) & (V - 1)
    level = torch.full((V,), -1, dtype=torch.int32, device="cuda")
    front = torch.zeros(V, dtype=torch.bool, device="cuda")
    front[ROOT] = True
    depth = 0
    while bool(front.any()):
        level[front] = depth
        new = torch.zeros_like(front)
        for d in DIFFS:
            new |= torch.roll(front, d)
        front = new & (level < 0)
        depth += 1
    torch.cuda.synchronize()
    yield p, off, col, level
    del off, col, level
    torch.cuda.empty_cache()


def _check(expect, lv, pa=None, st=None):
    torch.cuda.synchronize()
    assert torch.equal(lv, expect)
    if pa is not None:
        ids = torch.arange(V, device="cuda")
        assert int(pa[ROOT]) == ROOT and int(pa.min()) >= 0
        rest = ids != ROOT
        ok = torch.zeros(V, dtype=torch.bool, device="cuda")
        ok[torch.tensor(DIFFS, device="cuda")] = True
        assert bool((expect[pa.long()] == expect - 1)[rest].all())
        assert bool(ok[(ids - pa) % V][rest].all())
    if st is not None:
        assert (st.levels, st.reached, st.edges_scanned) == (int(expect.max()) + 1, V,
                                                             len(DIFFS) * V)


@pytest.mark.parametrize("dord", [0, 1])
def test_single_and_batch(graph, dord):
    p, off, col, expect = graph
    flags = p.BFS_WS_BATCH | (p.BFS_DEGREE_ORDER if dord else 0)
    ws = torch.empty(p.bfs_workspace_bytes(V, col.numel(), flags), dtype=torch.uint8, device="cuda")
    G = p.Graph(V, col.numel(), off, col, ws,
                p.bfs_graph_create(V, col.numel(), off, col, ws, flags=flags))
    for key, value in ((p.BFS_OPT_CLAIM_MODE, 1), (p.BFS_OPT_CLAIM_MODE, 0),
                       (p.BFS_OPT_FRONTIER_MODE, 1), (p.BFS_OPT_XCD_SLICES, 2),
                       (p.BFS_OPT_DIRECTION, 1)):
        print("case", dord, key, value, flush=True)
        saved = G.get_option(key)
        G.set_option(key, value)
        _check(expect, *G.run(ROOT))
        G.set_option(key, saved)
    rows, _ = G.run_batch([ROOT, 5, ROOT])
    _check(expect, rows[0].int())
    _check(expect, rows[2].int())
    _check(torch.roll(expect, 5 - ROOT), rows[1].int())
    G.close()


@pytest.mark.parametrize("R,C", [(1, 1), (2, 4)])
def test_blocked(graph, R, C):
    p, off, col, expect = graph
    n = p.bfs_grid2d_workspace_bytes(V, col.numel(), R, C)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    G = p.Grid2D(V, col.numel(), R, C, ws,
                 p.bfs_grid2d_create(V, col.numel(), off, col, R, C, ws, n))
    for mode in (0, 1, 2):
        print("case", R, C, mode, flush=True)
        _check(expect, *G.run(ROOT, msg_mode=mode))
    G.close()
