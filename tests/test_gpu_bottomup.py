"""Bottom-up steps against the oracle at the sizes where they change: units of
64 ids, a workgroup's 1024, ids on both sides of the 2^19 whose bits lie in
LDS, rows of no, one, four, five and very many neighbours, and lists of one
entry on a large graph."""
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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1_023, 1_025, 65_537, 524_287, 524_289, 700_001])
@pytest.mark.parametrize("dord", [0, 1])
def test_sizes(bfsmi, n, dord):
    rng = np.random.default_rng(n)
    m = 4 * n
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    keep = rng.random(m) < rng.random(m)  # some vertices without neighbours
    hub = np.full(n // 3, n - 1)
    src = np.concatenate([src[keep], hub, [n - 1]])
    dst = np.concatenate([dst[keep], rng.choice(n, size=n // 3, replace=False), [0]])
    g = graphgen.from_edges(n, src, dst)
    print("case", n, dord, flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    G.set_option(bfsmi.BFS_OPT_DIRECTION, 1)
    for alpha, beta, driver in ((14, 24, 0), (1000, 1000, 1), (1000, 1, 0)):
        G.set_option(bfsmi.BFS_OPT_DO_ALPHA, alpha)
        G.set_option(bfsmi.BFS_OPT_DO_BETA, beta)
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        for root in (n - 1, 0, n // 2):
            lv, pa, st = G.run(root)
            torch.cuda.synchronize()
            lv = lv.cpu().numpy()
            ref = oracle.bfs(g.off, g.col, root)
            assert np.array_equal(lv, ref.level)
            assert (st.levels, st.reached, st.edges_scanned) == (ref.nlevels, ref.reached,
                                                                 ref.edges_scanned)
            code, bad = oracle.validate(g.off, g.col, root, lv, pa.cpu().numpy())
            assert code == 0, (oracle.INVARIANTS[code], bad)
    G.close()
