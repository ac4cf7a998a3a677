"""Flag claims of the 2D blocked search against the oracle, at the edges of
their rule: blocks of one and of several bitmap words, ragged last blocks, a
level with one edge fewer, as many and one edge more than a processor's bitmap
has words, and grids in which some processors keep lists and others flag."""
import numpy as np
import pytest

import graphgen
from parity_util import assert_parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bfsmi():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1408_1605_amd as p
    p.load()
    return p


def _search(bfsmi, g, R, C, roots):
    G = bfsmi.Grid2D.from_csr(g.off, g.col, R, C)
    try:
        for mode in (0, 1, 2):
            print("case", g.name, R, C, mode, flush=True)
            items = []
            for r in roots:
                lv, pa, st = G.run(int(r), msg_mode=mode)
                torch.cuda.synchronize()
                items.append((int(r), lv.cpu().numpy(), pa.cpu().numpy(), st))
            assert_parity(g, items, label="%s %dx%d mode %d" % (g.name, R, C, mode))
    finally:
        G.close()


@pytest.mark.parametrize("R,C", [(1, 1), (1, 2), (4, 1), (2, 4), (8, 8)])
@pytest.mark.parametrize("n", [31, 257, 4_097, 70_003])
def test_dense_levels(bfsmi, R, C, n):
    rng = np.random.default_rng(n + R)
    g = graphgen.from_edges(n, rng.integers(0, n, 40 * n), rng.integers(0, n, 40 * n))
    g.name = "dense%d" % n
    _search(bfsmi, g, R, C, [0, n - 1])


@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_edge_count_at_the_rule(bfsmi, extra):
    # 1 x 1: the root's row has V / 32 + extra edges, the bitmap V / 32 words
    n = 32 * 64
    leaves = 64 + extra
    src = np.concatenate([np.zeros(leaves, np.int64), np.arange(1, leaves + 1)])
    dst = np.concatenate([np.arange(1, leaves + 1), np.arange(1, leaves + 1) + 1000])
    g = graphgen.from_edges(n, src, dst)
    g.name = "star%d" % leaves
    _search(bfsmi, g, 1, 1, [0])


@pytest.mark.parametrize("R,C", [(1, 8), (8, 1), (2, 4)])
def test_lists_beside_flags(bfsmi, R, C):
    # all heavy rows in one block: its processors flag, the others keep lists
    rng = np.random.default_rng(5)
    n = 16_384
    src = np.concatenate([rng.integers(0, 64, 60_000), rng.integers(0, n, 3_000)])
    dst = np.concatenate([rng.integers(0, n, 60_000), rng.integers(0, n, 3_000)])
    g = graphgen.from_edges(n, src, dst)
    g.name = "heavy%dx%d" % (R, C)
    _search(bfsmi, g, R, C, [1, n - 1, int(dst[-1])])


@pytest.mark.parametrize("leaves", [255, 257, 32_767, 32_769, 65_535, 65_536, 65_537])
@pytest.mark.parametrize("R,C", [(1, 1), (2, 4), (8, 8)])
def test_scan_widths(bfsmi, leaves, R, C):
    # the leaves' level: columns around a workgroup's 256 entries and levels
    # around the 65536 entries where a thread takes eight; 16 list units of
    # 2048 entries, above which plan and gather are two launches
    rng = np.random.default_rng(leaves)
    n = leaves + leaves // 2 + 7
    src = np.concatenate([np.zeros(leaves, np.int64), rng.integers(1, leaves + 1, leaves)])
    dst = np.concatenate([np.arange(1, leaves + 1), rng.integers(1, n, leaves)])
    g = graphgen.from_edges(n, src, dst)
    g.name = "leaves%d" % leaves
    _search(bfsmi, g, R, C, [0, 1])


@pytest.mark.parametrize("n", [1 << 24, (1 << 24) + 1])
def test_rows_at_the_rule(bfsmi, n):
    # 1 x 1: a level of more edges than bitmap words on both sides of the most
    # rows that are flagged
    leaves = n // 32 + 5
    rng = np.random.default_rng(3)
    leaf = rng.choice(n - 1, size=leaves, replace=False) + 1
    off = np.full(n + 1, 2 * leaves, np.int64)
    deg = np.zeros(n, np.int64)
    deg[0], deg[leaf] = leaves, 1
    off[0] = 0
    np.cumsum(deg, out=off[1:])
    col = np.zeros(2 * leaves, np.int32)
    col[:leaves] = np.sort(leaf)
    G = bfsmi.Grid2D.from_csr(off, col, 1, 1)
    try:
        for mode in (0, 2):
            print("case", n, mode, flush=True)
            lv, pa, st = G.run(0, msg_mode=mode)
            torch.cuda.synchronize()
            lv, pa = lv.cpu().numpy(), pa.cpu().numpy()
            exp = np.full(n, -1, np.int32)
            exp[0], exp[leaf] = 0, 1
            assert np.array_equal(lv, exp)
            exp[leaf] = 0
            assert np.array_equal(pa, exp)
            assert (st.levels, st.reached, st.edges_scanned) == (2, leaves + 1, 2 * leaves)
    finally:
        G.close()
