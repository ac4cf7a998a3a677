"""How the persistent loop decides to merge a level's claims, against the
oracle on both sides of each line: 65536 ids, degrees up to and above four
times the mean, symmetric and directed rows, levels of lattices and trees that
point at less and more than half of the ids; several merge levels in a row,
whose parents must not come from a stale bitmap; and workgroup shares around
1024 and 2048 vertices."""
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


def _uniform(n, mean, directed, top=0):
    # every id's row has `mean` edges; top: one row of that many more
    rng = np.random.default_rng(n + mean)
    src = np.concatenate([np.repeat(np.arange(n), mean), np.full(top, n // 2)])
    dst = rng.integers(0, n, src.size)
    return graphgen.from_edges(n, src, dst, symmetric=not directed)


def _cube(n):
    i = np.arange(n ** 3).reshape(n, n, n)
    src = np.concatenate([i[1:].ravel(), i[:, 1:].ravel(), i[:, :, 1:].ravel()])
    dst = np.concatenate([i[:-1].ravel(), i[:, :-1].ravel(), i[:, :, :-1].ravel()])
    return graphgen.from_edges(n ** 3, src, dst)


def _tree(fan, n):
    kid = np.arange(1, n)
    return graphgen.from_edges(n, (kid - 1) // fan, kid)


def _broad(leaves, spread):
    # root, 32 vertices, then leaves: the 32 share them evenly, or all but one
    # leaf each hang on the first
    at = 1 + (np.arange(leaves) % 32 if spread else np.minimum(np.arange(leaves)[::-1], 31))
    src = np.concatenate([np.zeros(32, np.int64), at])
    dst = np.concatenate([np.arange(1, 33), 33 + np.arange(leaves)])
    more = np.arange(33, 33 + leaves)  # one more level behind the leaves
    return graphgen.from_edges(33 + 2 * leaves, np.concatenate([src, more]),
                               np.concatenate([dst, more + leaves]))


CASES = {
    "uniform65536_2": lambda: _uniform(65_536, 2, False),
    "uniform65537_2": lambda: _uniform(65_537, 2, False),
    "uniform131072_4": lambda: _uniform(131_072, 4, False),
    "uniform200001_1": lambda: _uniform(200_001, 1, False),
    "hub131072_4": lambda: _uniform(131_072, 4, False, top=60),  # one row in 131,072 above 4 x 8
    "directed65536_3": lambda: _uniform(65_536, 3, True),
    "directed65537_3": lambda: _uniform(65_537, 3, True),
    "directed200001_5": lambda: _uniform(200_001, 5, True),
    "directedhub200001_5": lambda: _uniform(200_001, 5, True, top=16),
    "cube40": lambda: _cube(40), "cube41": lambda: _cube(41),
    "tree3_9841": lambda: _tree(3, 9_841), "tree2_8191": lambda: _tree(2, 8_191),
    "tree2_65535": lambda: _tree(2, 65_535), "grid40x50": lambda: graphgen.grid(40, 50),
    "even32736": lambda: _broad(32 * 1_023, True), "even32768": lambda: _broad(32 * 1_024, True),
    "even32800": lambda: _broad(32 * 1_025, True), "even65536": lambda: _broad(32 * 2_048, True),
    "uneven2047": lambda: _broad(2_047, False), "uneven2080": lambda: _broad(2_080, False),
    "uneven8000": lambda: _broad(8_000, False),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_merge_lines(bfsmi, case):
    g = CASES[case]()
    directed = case.startswith("directed")
    print("case", case, "V=%d nnz=%d" % (g.V, g.nnz), flush=True)
    roots = [0, g.V - 1, g.V // 2]
    refs = [oracle.bfs(g.off, g.col, r) for r in roots]

    def check(lv, pa, st, ref, root):
        torch.cuda.synchronize()
        lv = lv.cpu().numpy()
        assert np.array_equal(lv, ref.level)
        assert (st.levels, st.reached, st.edges_scanned) == (ref.nlevels, ref.reached,
                                                             ref.edges_scanned)
        code, bad = oracle.validate(g.off, g.col, root, lv, pa.cpu().numpy(), directed=directed)
        assert code == 0, (oracle.INVARIANTS[code], bad)

    for flags in (0, bfsmi.BFS_DEGREE_ORDER):
        G = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
        for r, ref in zip(roots, refs):
            lv, pa, st = G.run(r)
            check(lv, pa, st, ref, r)
        if flags == 0:
            for r, ref in zip(roots, refs):
                lv, pa = torch.empty_like(lv), torch.empty_like(pa)
                st = bfsmi.bfs_run_noalloc(G.V, G.nnz, G.off, G.col, r, lv, pa)
                check(lv, pa, st, ref, r)
        G.close()
