"""The edge counts of the direction-optimizing mode on graphs whose frontier
grows slowly: several top-down levels in bitmap form before the switch (and
after the switch back), on workspaces of any contents, many roots on one
handle.  Levels and edges_scanned against the oracle."""
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


def _uniform(n):
    # mean degree 8: eight times the vertices every level
    rng = np.random.default_rng(n)
    return graphgen.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n))


def _tree(depth):
    # binary, its leaves joined pairwise to a second tree, mirrored: the
    # frontier doubles, then halves
    n = (1 << (depth + 1)) - 1
    i = np.arange(1, n)
    leaf = np.arange((n - 1) // 2, n)
    return graphgen.from_edges(2 * n, np.concatenate([(i - 1) // 2, n + (i - 1) // 2, leaf]),
                               np.concatenate([i, n + i, n + leaf]))


GRAPHS = {"uniform30001": lambda: _uniform(30_001), "uniform300000": lambda: _uniform(300_000),
          "tree15": lambda: _tree(15)}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("dord", [0, 1])
@pytest.mark.parametrize("fill", [0x00, 0xff])
def test_edges_of_a_slow_frontier(bfsmi, name, dord, fill):
    g = GRAPHS[name]()
    print("case", name, dord, fill, flush=True)
    flags = bfsmi.BFS_DEGREE_ORDER if dord else 0
    off, col = torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda()
    ws = torch.full((bfsmi.bfs_workspace_bytes(g.V, g.nnz, flags),), fill, dtype=torch.uint8,
                    device="cuda")
    torch.cuda.synchronize()
    G = bfsmi.Graph(g.V, g.nnz, off, col, ws,
                    bfsmi.bfs_graph_create(g.V, g.nnz, off, col, ws, flags=flags))
    roots = [0, g.V - 1, g.V // 3]
    refs = [oracle.bfs(g.off, g.col, r) for r in roots]
    G.set_option(bfsmi.BFS_OPT_DIRECTION, 1)
    G.set_option(bfsmi.BFS_OPT_LOOP_LIMIT, 64)
    steps = 0
    for alpha, beta, driver, mode in ((14, 24, 0, 0), (1, 24, 1, 2), (1, 24, 0, 0), (2, 2, 1, 0),
                                      (4, 1, 1, 2)):
        G.set_option(bfsmi.BFS_OPT_DO_ALPHA, alpha)
        G.set_option(bfsmi.BFS_OPT_DO_BETA, beta)
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        for root, ref in zip(roots, refs):
            lv, _, st = G.run(root)
            torch.cuda.synchronize()
            assert np.array_equal(lv.cpu().numpy(), ref.level)
            assert (st.levels, st.reached, st.edges_scanned) == (
                ref.nlevels, ref.reached, ref.edges_scanned), (alpha, beta, driver, mode, root)
            steps += st.bottom_up_levels
    assert steps > 0
    G.close()
