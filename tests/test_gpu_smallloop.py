"""The persistent small-level loop against the oracle, at the sizes where it
changes its way: workgroup shares that fill exactly (32 x 1024 vertices),
overflow into the queue or go back to the host; rows of at most four edges
(one lane per edge) and of more (mapped tiles); hub rows on both sides of the
hot id range (65536); and searches on several handles at the same time, whose
workgroups have to start together."""
import threading

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


def _tree(fan, n):
    """The first n vertices of a complete fan-ary tree, ids breadth-first."""
    kid = np.arange(1, n, dtype=np.int64)
    g = graphgen.from_edges(n, (kid - 1) // fan, kid)
    g.name = "tree%d_%d" % (fan, n)
    return g


def _triangles(w, h):
    """Grid with one diagonal per cell: rows of up to six edges."""
    ids = np.arange(w * h, dtype=np.int64).reshape(h, w)
    src = [ids[:, :-1].ravel(), ids[:-1, :].ravel(), ids[:-1, :-1].ravel()]
    dst = [ids[:, 1:].ravel(), ids[1:, :].ravel(), ids[1:, 1:].ravel()]
    g = graphgen.from_edges(w * h, np.concatenate(src), np.concatenate(dst))
    g.name = "triangles%dx%d" % (w, h)
    return g


def _hubs(n, hubs, degree):
    """hubs vertices of the given degree spread over n ids, on a path."""
    rng = np.random.default_rng(hubs)
    at = rng.choice(n, size=hubs, replace=False)
    src = [np.repeat(at, degree), np.arange(n - 1)]
    dst = [rng.integers(0, n, hubs * degree), np.arange(1, n)]
    g = graphgen.from_edges(n, np.concatenate(src), np.concatenate(dst))
    g.name = "hubs%d_%d" % (n, hubs)
    return g


CASES = {
    "tree2_32767": lambda: (_tree(2, (1 << 15) - 1), [0, 3, 20_000]),
    "tree2_65535": lambda: (_tree(2, (1 << 16) - 1), [0]),      # shares exactly full
    "tree2_131071": lambda: (_tree(2, (1 << 17) - 1), [0, 1]),  # 65536 leaves: shares overflow
    "tree2_300000": lambda: (_tree(2, 300_000), [0]),           # a frontier over the limit
    "tree3_100001": lambda: (_tree(3, 100_001), [0, 99_999]),
    "tree5_200003": lambda: (_tree(5, 200_003), [0, 7]),
    "grid301x57": lambda: (graphgen.grid(301, 57), [0, 150 + 28 * 301]),
    "triangles257x131": lambda: (_triangles(257, 131), [0, 128 + 65 * 257]),
    "hubs70001": lambda: (_hubs(70_001, 30, 800), [0, 69_000]),
    "hubs3001": lambda: (_hubs(3_001, 3, 2_000), [0]),
    "path2": lambda: (graphgen.from_edges(2, [0], [1]), [0, 1]),
    "alone": lambda: (graphgen.from_edges(1, np.zeros(0), np.zeros(0)), [0]),
}


def _check(g, G, root, want_parents=True):
    lv, pa, st = G.run(int(root), want_parents=want_parents)
    torch.cuda.synchronize()
    lv = lv.cpu().numpy()
    ref = oracle.bfs(g.off, g.col, int(root))
    assert np.array_equal(lv, ref.level)
    assert (st.levels, st.reached, st.edges_scanned) == (ref.nlevels, ref.reached,
                                                         ref.edges_scanned)
    if want_parents:
        code, bad = oracle.validate(g.off, g.col, int(root), lv, pa.cpu().numpy())
        assert code == 0, (oracle.INVARIANTS[code], bad)
    return st


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("dord", [0, 1])
def test_small_loop(bfsmi, case, dord):
    g, roots = CASES[case]()
    print("case", case, dord, "V=%d nnz=%d" % (g.V, g.nnz), flush=True)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    for r in roots:
        st = _check(g, G, r)
        assert st.device_loop_levels > 0
        _check(g, G, r, want_parents=False)
    # a low frontier limit: the loop hands back and takes over again
    G.set_option(bfsmi.BFS_OPT_LOOP_LIMIT, 64)
    for r in roots:
        _check(g, G, r)
    G.close()


def test_small_loop_many_handles_at_once(bfsmi):
    # twenty handles, so every XCD runs the loops of more than one
    g = graphgen.grid(160, 90)
    roots = [0, 77, g.V - 1, g.V // 2]
    refs = {r: oracle.bfs(g.off, g.col, r).level for r in roots}
    handles = [bfsmi.Graph.from_csr(g.off, g.col) for _ in range(20)]
    streams = [torch.cuda.Stream() for _ in handles]
    bad = []

    def client(G, s):
        for k in range(6):
            r = roots[k % len(roots)]
            with torch.cuda.stream(s):
                lv, _, _ = G.run(r, stream=s)
                s.synchronize()
                if not np.array_equal(lv.cpu().numpy(), refs[r]):
                    bad.append(r)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=client, args=a) for a in zip(handles, streams)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for G in handles:
        G.close()
