"""The persistent serving levels against the oracle where they change their
way: graphs on one workgroup and just above, rows of at most four edges and
longer ones, shares that overflow or grow uneven and are dealt out anew, hubs
at and over the degree limit, and vertices without out-edges."""
import time

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


def _path(n):
    return graphgen.from_edges(n, np.arange(n - 1), np.arange(1, n))


def _broom(leaves):
    # a path of 80, then a hub
    src = np.concatenate([np.arange(79), np.full(leaves, 79)])
    return graphgen.from_edges(80 + leaves, src, np.arange(1, 80 + leaves))


def _tree(depth):
    # a path of 60, then a binary tree: its levels double
    n = (1 << (depth + 1)) - 1
    i = np.arange(1, n)
    src = np.concatenate([np.arange(60), 60 + (i - 1) // 2])
    dst = np.concatenate([np.arange(1, 61), 60 + i])
    return graphgen.from_edges(60 + n, src, dst)


def _diagonal_grid(side):
    i = np.arange(side * side).reshape(side, side)
    src = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel(), i[:-1, :-1].ravel()])
    dst = np.concatenate([i[:, 1:].ravel(), i[1:].ravel(), i[1:, 1:].ravel()])
    return graphgen.from_edges(side * side, src, dst)


def _one_way(n):
    # out-edges only, with loops and shortcuts; the last vertex has none
    rng = np.random.default_rng(2)
    i = np.arange(n - 1)
    s = rng.integers(0, n - 9, n)
    src, dst = np.concatenate([i, i, s]), np.concatenate([i + 1, i, s + rng.integers(1, 9, n)])
    return graphgen.from_edges(n, src, dst, symmetric=False)


CASES = {
    "path100": lambda: _path(100), "path127": lambda: _path(127), "path128": lambda: _path(128),
    "path129": lambda: _path(129), "path3000": lambda: _path(3000),
    "broom5000": lambda: _broom(5000), "broom9000": lambda: _broom(9000),
    "tree10": lambda: _tree(10), "tree16": lambda: _tree(16),
    "diagonal150": lambda: _diagonal_grid(150), "oneway2000": lambda: _one_way(2000),
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("dord", [0, 1])
def test_serving_levels(bfsmi, case, dord):
    g = CASES[case]()
    print("case", case, dord, "V=%d" % g.V, flush=True)
    h = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    arena = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    s = bfsmi.bfs_server_create(arena, max_lanes=64, max_inflight=4, flags=0)
    gid = bfsmi.bfs_server_add_graph(s, h.handle)
    rng = np.random.default_rng(g.V)
    # the first queries teach the server that the graph is deep
    waves = [[0, 1], [0] + [int(r) for r in rng.integers(0, g.V, 11)], [g.V - 1, 0, 1]]
    for roots in waves:
        ts = [bfsmi.bfs_submit(s, gid, r) for r in roots]
        end = time.time() + 30
        left = set(ts)
        while left and time.time() < end:
            left -= set(bfsmi.bfs_server_completed(s))
            time.sleep(1e-4)
        assert not left
        for t, r in zip(ts, roots):
            got = np.empty(g.V, dtype=np.int32)
            code, _ = bfsmi.bfs_poll(s, t, got)
            assert code == bfsmi.BFS_OK
            assert np.array_equal(got, oracle.bfs(g.off, g.col, r).level), r
    st = bfsmi.bfs_server_get_stats(s)
    assert st.failed == 0 and st.persistent_rounds > 0
    bfsmi.bfs_server_destroy(s)
    h.close()
