"""Batch levels searched from the unseen side (degree-ordered, symmetric
graphs) against the oracle: every row equal element by element, and the
union search's counts equal to those of the oracle's rows.

The graphs have rows on both sides of every cut the kernel makes (32, 256 and
4096 edges, and hub rows cut into pieces of 2048), vertex counts that leave
partial waves, and a tail whose end joins the dense part late, so that some
lanes are expanded while others are searched from the unseen side."""
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


def _hubs(n, degrees, extra, tail, seed):
    """Random symmetric graph on n vertices: vertex i < len(degrees) gets
    degrees[i] random neighbours, extra random edges on top, a path of tail
    vertices hanging off vertex 0, and three isolated vertices."""
    rng = np.random.default_rng(seed)
    src = [np.full(d, i, np.int64) for i, d in enumerate(degrees)]
    dst = [rng.choice(n, size=d, replace=False) for d in degrees]
    src.append(rng.integers(0, n, extra))
    dst.append(rng.integers(0, n, extra))
    chain = np.concatenate([[0], np.arange(n, n + tail)])
    src.append(chain[:-1])
    dst.append(chain[1:])
    g = graphgen.from_edges(n + tail + 3, np.concatenate(src), np.concatenate(dst))
    g.name = "hubs%d" % n
    return g


def _union_counts(g, rows):
    deg = np.diff(g.off)
    reached = edges = 0
    for d in range(int(rows.max()) + 1):
        front = (rows == d).any(axis=0)
        reached += int(front.sum())
        edges += int(deg[front].sum())
    return int(rows.max()) + 1, reached, edges


CASES = {
    "cuts": lambda: _hubs(20_011, [31, 32, 33, 255, 256, 257, 2047, 4095, 4096, 4097, 6144, 12_000],
                          40_000, 9, 1),
    "hubs": lambda: _hubs(9_001, [8000] * 70 + [300] * 40, 3_000, 30, 2),
    "no_hubs": lambda: _hubs(5_003, [40] * 100, 20_000, 5, 3),
    "rmat": lambda: graphgen.rmat(15),
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("n_roots", [1, 5, 64])
def test_batch_pull_levels(bfsmi, case, n_roots):
    g = CASES[case]()
    print("case", case, "V=%d nnz=%d roots=%d" % (g.V, g.nnz, n_roots), flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_WS_BATCH | bfsmi.BFS_DEGREE_ORDER)
    picks = [int(r) for r in graphgen.pick_roots(g, 64, 17)]
    # the tail's end and an isolated vertex among them
    roots = ([g.V - 4, g.V - 1] + picks)[:n_roots] if n_roots > 1 else picks[:1]
    exp = oracle.batch_levels_int8(g.off, g.col, roots)
    counts = _union_counts(g, exp)
    for driver in (0, 1, 0):
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        got, st = G.run_batch(roots)
        torch.cuda.synchronize()
        bad = np.nonzero((got.cpu().numpy() != exp).any(axis=1))[0]
        assert bad.size == 0, (driver, bad[:8])
        assert (st.levels, st.reached, st.edges_scanned) == counts
    G.close()


def test_batch_directed_graph_keeps_out_edges(bfsmi):
    # a CSR that is not its own transpose: no level may read rows as in-edges
    rng = np.random.default_rng(4)
    n = 6_000
    src, dst = rng.integers(0, n, 90_000), rng.integers(0, n, 90_000)
    g = graphgen.from_edges(n, src, dst, symmetric=False)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_WS_BATCH | bfsmi.BFS_DEGREE_ORDER)
    roots = [int(r) for r in graphgen.pick_roots(g, 20, 3)]
    exp = oracle.batch_levels_int8(g.off, g.col, roots)
    got, _ = G.run_batch(roots)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), exp)
    G.close()
