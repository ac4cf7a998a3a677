"""One-launch level scans (k_list_scan, k_front_scan) against the oracle where
they change their way: vertex counts around the groups of 8 ids, the blocks of
2048 and (above 2^19 vertices) 8192 ids, lists on both sides of 65536 entries,
rows of no, few and very many edges, every tile size, with and without the
row prefix skip, and row offsets that allow no 16-byte loads."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bfsmi():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1408_1605_amd as p
    p.load()
    return p


def _check(g, G, root, directed=False, rows_sorted=True):
    lv, pa, st = G.run(int(root))
    torch.cuda.synchronize()
    lv = lv.cpu().numpy()
    ref = oracle.bfs(g.off, g.col, int(root))
    assert np.array_equal(lv, ref.level)
    assert (st.levels, st.reached, st.edges_scanned) == (ref.nlevels, ref.reached,
                                                         ref.edges_scanned)
    code, bad = oracle.validate(g.off, g.col, int(root), lv, pa.cpu().numpy(), directed=directed,
                                rows_sorted=rows_sorted)
    assert code == 0, (oracle.INVARIANTS[code], bad)
    return st


def _random(n, m, seed, hub=0):
    rng = np.random.default_rng(seed)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    if hub:
        src = np.concatenate([src, np.full(hub, n // 3)])
        dst = np.concatenate([dst, rng.choice(n, size=hub, replace=False)])
    g = graphgen.from_edges(n, src, dst)
    g.name = "random%d" % n
    return g


@pytest.mark.parametrize("n", [7, 8, 9, 2047, 2048, 2049, 16_391, 70_003, 140_001])
@pytest.mark.parametrize("dord", [0, 1])
def test_sizes(bfsmi, n, dord):
    g = _random(n, 8 * n, n, hub=n // 2)
    print("case", g.name, dord, flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    root = int(np.argmax(np.diff(g.off)))
    for driver, mode, ept in ((0, 0, 4), (1, 0, 4), (1, 2, 1), (1, 2, 8), (1, 1, 2)):
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        G.set_option(bfsmi.BFS_OPT_EDGES_PER_THREAD, ept)
        for r in (root, 0, n - 1):
            _check(g, G, r)
    G.close()


@pytest.mark.parametrize("n", [524_287, 524_288, 524_289, 532_481, 600_003])
@pytest.mark.parametrize("dord", [0, 1])
def test_block_widths(bfsmi, n, dord):
    # bitmap levels on both sides of the wide blocks' line, last blocks of one
    # and of many ids
    g = _random(n, 3 * n, n, hub=n // 2)
    print("case", g.name, dord, flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, 1)
    for mode in (0, 2):
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        _check(g, G, int(np.argmax(np.diff(g.off))))
    G.close()


@pytest.mark.parametrize("leaves", [65_535, 65_536, 65_537, 200_003])
def test_list_lengths(bfsmi, leaves):
    # the leaves' level is a list (mode 1) of that many entries
    n = 2 * leaves + 1
    kid = np.arange(1, n, dtype=np.int64)
    g = graphgen.from_edges(n, np.where(kid <= leaves, 0, kid - leaves), kid)
    G = bfsmi.Graph.from_csr(g.off, g.col)
    G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, 1)
    for mode in (0, 1):
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        _check(g, G, 0)
        _check(g, G, n - 1)
    G.close()


@pytest.mark.parametrize("skip", [0, 1])
@pytest.mark.parametrize("summary", [0, 1, 2])
def test_prefix_skip(bfsmi, skip, summary):
    g = graphgen.rmat(18)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER)
    G.set_option(bfsmi.BFS_OPT_ROW_SKIP, skip)
    G.set_option(bfsmi.BFS_OPT_VISITED_SUMMARY, summary)
    for xs in (0, 1, 2):
        G.set_option(bfsmi.BFS_OPT_XCD_SLICES, xs)
        for r in graphgen.pick_roots(g, 2, 5):
            st = _check(g, G, r)
            assert st.edges_examined <= st.edges_scanned
            if not (skip and summary):
                assert st.edges_examined == st.edges_scanned
    G.close()


def test_directed_rows_without_edges(bfsmi):
    rng = np.random.default_rng(8)
    n = 90_000
    src = np.concatenate([np.zeros(60_000, np.int64), rng.integers(1, 400, 300_000)])
    dst = np.concatenate([rng.choice(n, 60_000, replace=False), rng.integers(0, n, 300_000)])
    g = graphgen.from_edges(n, src, dst, symmetric=False)
    for flags in (0, bfsmi.BFS_DEGREE_ORDER):
        G = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
        for driver in (0, 1):
            G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
            _check(g, G, 0, directed=True)
        G.close()


def test_row_offsets_at_odd_address(bfsmi):
    # the caller's offsets need only 8-byte alignment
    g = _random(30_001, 200_000, 12, hub=9_000)
    room = torch.empty(g.V + 2, dtype=torch.int64, device="cuda")
    off = room[1:]
    off.copy_(torch.from_numpy(g.off))
    assert off.data_ptr() % 16 == 8
    col = torch.from_numpy(g.col).cuda()
    need = bfsmi.bfs_workspace_bytes(g.V, g.nnz, 0)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    G = bfsmi.Graph(g.V, g.nnz, off, col, ws,
                    bfsmi.bfs_graph_create(g.V, g.nnz, off, col, ws, need, 0))
    G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, 1)
    for mode in (0, 2):
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        _check(g, G, 17)
    G.close()


def test_wide_blocks_above_2_24_vertices(bfsmi):
    # star of stars on 2^24 + 4099 vertices: dense levels in 8192-id blocks
    n = (1 << 24) + 4099
    kid = np.arange(1, n, dtype=np.int64)
    up = np.where(kid <= 3000, 0, (kid * 2654435761) % 3000 + 1)
    order = np.argsort(np.concatenate([up, kid]), kind="stable")
    src = np.concatenate([up, kid])[order]
    dst = np.concatenate([kid, up])[order]
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=off[1:])
    g = graphgen.CSR(off, dst.astype(np.int32), name="stars")
    for flags in (0, bfsmi.BFS_DEGREE_ORDER):
        G = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
        for r in (0, n - 1):
            _check(g, G, r, rows_sorted=False)  # (built in order of kid, then of up)
        G.close()
