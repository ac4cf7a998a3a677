"""The batch's one-launch degree scans against the oracle: queues on both sides
of one workgroup's 256 entries, of a chunk of 2048 vertices and of the 131072
entries above which a workgroup takes 2048, scanned from the queue (degree
order; single levels) and by the finalize of the level before; graphs on both
sides of the 2^17 and 2^18 vertices where the finalize changes its chunks and
levels may be sparse."""
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


def _union_counts(g, rows):
    deg = np.diff(g.off)
    reached = edges = 0
    for d in range(int(rows.max()) + 1):
        front = (rows == d).any(axis=0)
        reached += int(front.sum())
        edges += int(deg[front].sum())
    return int(rows.max()) + 1, reached, edges


# a hub with n leaves, a third of them with a few edges more: its level is a
# queue of n entries, many of degree 1
@pytest.mark.parametrize("leaves", [1, 255, 256, 257, 2_047, 2_048, 2_049, 65_533, 65_535, 90_001, 131_067,
                                    131_071, 131_073, 300_007])
@pytest.mark.parametrize("dord", [0, 1])
@pytest.mark.parametrize("symmetric", [True, False])
def test_queue_lengths(bfsmi, leaves, dord, symmetric):
    rng = np.random.default_rng(leaves)
    n = 2 * leaves + 5
    extra = leaves // 3
    src = np.concatenate([np.zeros(leaves, np.int64), rng.integers(1, leaves + 1, 3 * extra)])
    dst = np.concatenate([np.arange(1, leaves + 1), rng.integers(1, n, 3 * extra)])
    g = graphgen.from_edges(n, src, dst, symmetric=symmetric)
    print("case", leaves, dord, symmetric, flush=True)
    flags = bfsmi.BFS_WS_BATCH | (bfsmi.BFS_DEGREE_ORDER if dord else 0)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
    roots = [0, 1, leaves, n - 1]
    exp = oracle.batch_levels_int8(g.off, g.col, roots)
    counts = _union_counts(g, exp)
    for driver, tile in ((0, 1024), (1, 256), (0, 2048)):
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        G.set_option(bfsmi.BFS_OPT_BATCH_TILE, tile)
        got, st = G.run_batch(roots)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), exp)
        assert (st.levels, st.reached, st.edges_scanned) == counts
    G.close()
