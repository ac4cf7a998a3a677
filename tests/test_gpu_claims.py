"""Claims of graphs without degree order (BFS_OPT_CLAIM_MODE): the byte flags
share the degree array, so searches that use it for degrees (the direction-
optimizing mode, batches) run between flag searches on the same handle."""
from types import SimpleNamespace

import numpy as np
import pytest

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


def _check(g, G, root, directed, parents=True):
    lv, pa, st = G.run(int(root), want_parents=parents)
    torch.cuda.synchronize()
    lv = lv.cpu().numpy()
    ref = oracle.bfs(g.off, g.col, int(root))
    assert np.array_equal(lv, ref.level)
    assert (st.reached, st.edges_scanned) == (ref.reached, ref.edges_scanned)
    if parents:
        code, bad = oracle.validate(g.off, g.col, int(root), lv, pa.cpu().numpy(),
                                    directed=directed, rows_sorted=False)
        assert code == 0, (oracle.INVARIANTS[code], bad)


# 1..9: the flags (32 bytes a word) are longer than V degrees and end in the
# region's padding; 33, 65_535: a last word with one and with 31 ids
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 32, 33, 65_535, 200_001])
@pytest.mark.parametrize("directed", [False, True])
def test_plain_claims(bfsmi, n, directed):
    rng = np.random.default_rng(n)
    m = 12 * n
    src, dst = rng.integers(0, n, m), (rng.integers(0, n, m) * rng.random(m)).astype(np.int64)
    if not directed:
        src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    order = np.argsort(src, kind="stable")  # loops and multi-edges stay
    off = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    g = SimpleNamespace(off=off, col=dst[order].astype(np.int32))
    print("case", n, directed, flush=True)
    G = bfsmi.Graph.from_csr(off, g.col, flags=bfsmi.BFS_WS_BATCH)
    root = int(np.argmax(np.diff(off)))
    for claim in (2, 0, 1, 2):
        G.set_option(bfsmi.BFS_OPT_CLAIM_MODE, claim)
        for driver, mode in ((1, 2), (1, 0), (0, 0)):
            G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
            G.set_option(bfsmi.BFS_OPT_FRONTIER_MODE, mode)
            for r in (root, 0, n - 1):
                _check(g, G, r, directed, parents=claim != 1)
        if not directed:
            G.set_option(bfsmi.BFS_OPT_DIRECTION, 1)
            _check(g, G, root, directed)
            G.set_option(bfsmi.BFS_OPT_DIRECTION, 0)
        roots = [root, 0, n - 1]
        got, _ = G.run_batch(roots)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.batch_levels_int8(off, g.col, roots))
    G.close()
