"""The one-launch scan of XCD-sliced levels against the oracle: frontiers around
a workgroup's 256 entries, slices that share nothing but the tile sizes, hot
ids dealt by row, and a graph whose tiles of 256 edges leave no room for the
slices' own (which takes the four-launch scan)."""
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


@pytest.mark.parametrize("leaves", [1, 255, 256, 257, 2_000])
@pytest.mark.parametrize("n", [17_003, 70_001])
def test_sliced_frontiers(bfsmi, n, leaves):
    # root - leaves - the rest: the leaves' level is the sliced one
    rng = np.random.default_rng(n + leaves)
    root = n - 1
    leaf = rng.choice(n - 1, size=leaves, replace=False)
    m = 20_000
    src = np.concatenate([np.full(leaves, root), leaf[rng.integers(0, leaves, m)],
                          rng.integers(0, n, n // 4)])
    dst = np.concatenate([leaf, rng.integers(0, n, m), rng.integers(0, n, n // 4)])
    g = graphgen.from_edges(n, src, dst)
    print("case", n, leaves, flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER)
    G.set_option(bfsmi.BFS_OPT_XCD_SLICES, 2)
    for driver, ept, mode in ((1, 4, 0), (1, 1, 2), (0, 8, 0), (1, 2, 1)):
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        G.set_option(bfsmi.BFS_OPT_EDGES_PER_THREAD, ept)
        G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
        for r in (root, int(leaf[0]), root):
            lv, pa, st = G.run(r)
            torch.cuda.synchronize()
            lv = lv.cpu().numpy()
            ref = oracle.bfs(g.off, g.col, r)
            assert np.array_equal(lv, ref.level)
            assert (st.levels, st.reached, st.edges_scanned) == (ref.nlevels, ref.reached,
                                                                 ref.edges_scanned)
            code, bad = oracle.validate(g.off, g.col, r, lv, pa.cpu().numpy())
            assert code == 0, (oracle.INVARIANTS[code], bad)
    G.close()
