"""The scans of graphs of 2^32 edges and more, on small graphs: a handle whose
limit has been lowered searches with the kernels that number a level's edges in
64 bits.  Every entry point against the oracle, and its counts against a handle
that scans its levels in one launch."""
import ctypes
import time

import numpy as np
import pytest

import graphgen
import oracle
from parity_util import assert_parity, gpu_results

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bfsmi():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1408_1605_amd as p
    p.load()
    return p


def _lower(bfsmi, name, handle):
    f = getattr(bfsmi.load(), name)
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int64]
    assert f(handle, 0) == bfsmi.BFS_OK
    assert f(handle, 1) == bfsmi.BFS_ERR_INVALID  # not raised again


def _hub(n):
    # a row of many tiles, and as many entries without out-edges at its end
    rng = np.random.default_rng(n)
    src = np.concatenate([np.zeros(n - 1, np.int64), rng.integers(1, n // 2, 3 * n)])
    dst = np.concatenate([np.arange(1, n), rng.integers(1, n, 3 * n)])
    g = graphgen.from_edges(n, src, dst, symmetric=False)
    g.name = "hub%d" % n
    return g


def _rmat(scale):
    g = graphgen.rmat(scale)
    g.name = "rmat%d" % scale
    return g


GRAPHS = {"rmat12": lambda: _rmat(12), "rmat18": lambda: _rmat(18), "hub50021": lambda: _hub(50_021),
          "grid90": lambda: graphgen.grid(90)}


def _roots(g, n):
    return [0] + [int(r) for r in graphgen.pick_roots(g, n, 5)]


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("dord", [0, 1])
def test_single(bfsmi, name, dord):
    g = GRAPHS[name]()
    flags = bfsmi.BFS_DEGREE_ORDER if dord else 0
    A = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
    B = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
    _lower(bfsmi, "bfs_test_pack_limit", A.handle)
    roots = _roots(g, 2)
    O = bfsmi
    for opts in ({}, {O.BFS_OPT_LOOP_DRIVER: 1}, {O.BFS_OPT_LOOP_DRIVER: 1, O.BFS_OPT_FRONTIER_MODE: 1},
                 {O.BFS_OPT_LOOP_DRIVER: 1, O.BFS_OPT_FRONTIER_MODE: 2, O.BFS_OPT_CLAIM_MODE: 0},
                 {O.BFS_OPT_LOOP_LIMIT: 64, O.BFS_OPT_CLAIM_MODE: 2, O.BFS_OPT_XCD_SLICES: 2},
                 {O.BFS_OPT_LOOP_DRIVER: 1, O.BFS_OPT_XCD_SLICES: 2, O.BFS_OPT_EDGES_PER_THREAD: 1},
                 {O.BFS_OPT_LOOP_LIMIT: 64, O.BFS_OPT_VISITED_SUMMARY: 1},
                 {O.BFS_OPT_LOOP_DRIVER: 1, O.BFS_OPT_ROW_SKIP: 0, O.BFS_OPT_EDGES_PER_THREAD: 8}):
        print("case", name, dord, opts, flush=True)
        saved = {k: A.get_option(k) for k in opts}
        for G in (A, B):
            for k, v in opts.items():
                G.set_option(k, v)
        a, b = gpu_results(torch, A, roots), gpu_results(torch, B, roots)
        assert_parity(g, a, directed=name.startswith("hub"), label="%s wide" % name)
        for x, y in zip(a, b):
            assert (x[3].bitmap_levels, x[3].expand_launches) == (y[3].bitmap_levels,
                                                                  y[3].expand_launches)
        for G in (A, B):
            for k, v in saved.items():
                G.set_option(k, v)
    A.close()
    B.close()


@pytest.mark.parametrize("dord", [0, 1])
def test_direction(bfsmi, dord):
    g = _rmat(16)
    G = bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0)
    _lower(bfsmi, "bfs_test_pack_limit", G.handle)
    G.set_option(bfsmi.BFS_OPT_DIRECTION, 1)
    for alpha, driver in ((14, 0), (1, 1), (1000, 1)):
        G.set_option(bfsmi.BFS_OPT_DO_ALPHA, alpha)
        G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        assert_parity(g, gpu_results(torch, G, _roots(g, 2)), label="rmat16 wide alpha %d" % alpha)
    G.close()


@pytest.mark.parametrize("name", sorted(GRAPHS) + ["rmat19"])  # above 2^18: sparse levels too
@pytest.mark.parametrize("dord", [0, 1])
def test_batch(bfsmi, name, dord):
    g = GRAPHS[name]() if name in GRAPHS else _rmat(19)
    flags = bfsmi.BFS_WS_BATCH | (bfsmi.BFS_DEGREE_ORDER if dord else 0)
    A = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
    B = bfsmi.Graph.from_csr(g.off, g.col, flags=flags)
    one = [g.V // 2] * (64 if name == "rmat18" else 5)
    if name == "grid90":  # its corners are deeper than a batch goes
        batches = [[45 * 90 + 45, 45 * 90 + 44, 30 * 90 + 60], [45 * 90 + 45]]
    else:
        batches = [_roots(g, len(one) - 1), one, _roots(g, 1)]
    A.run_batch(batches[0])  # captured before the limit changes
    torch.cuda.synchronize()
    _lower(bfsmi, "bfs_test_pack_limit", A.handle)
    for driver in (0, 1):
        for G in (A, B):
            G.set_option(bfsmi.BFS_OPT_LOOP_DRIVER, driver)
        for roots in batches:
            print("case", name, dord, driver, len(roots), flush=True)
            got, st = A.run_batch(roots)
            ref, sb = B.run_batch(roots)
            torch.cuda.synchronize()
            exp = oracle.batch_levels_int8(g.off, g.col, roots)
            assert np.array_equal(got.cpu().numpy(), exp)
            assert np.array_equal(ref.cpu().numpy(), exp)
            assert (st.levels, st.reached, st.edges_scanned) == (sb.levels, sb.reached,
                                                                 sb.edges_scanned)
    A.close()
    B.close()


@pytest.mark.parametrize("dord", [0, 1])
def test_serving(bfsmi, dord):
    gs = [_rmat(14), graphgen.grid(70), _hub(3_001)]
    hs = [bfsmi.Graph.from_csr(g.off, g.col, flags=bfsmi.BFS_DEGREE_ORDER if dord else 0) for g in gs]
    for h in hs:
        _lower(bfsmi, "bfs_test_pack_limit", h.handle)
    arena = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    # without persistent rounds, so that every level is one of the scanned ones
    s = bfsmi.bfs_server_create(arena, flags=bfsmi.BFS_SRV_NO_PERSISTENT)
    ids = [bfsmi.bfs_server_add_graph(s, h.handle) for h in hs]
    for wave in range(2):
        jobs = [(k, int(r)) for k, g in enumerate(gs)
                for r in np.random.default_rng(wave).integers(0, g.V, 9)]
        print("case", dord, wave, flush=True)
        ts = [bfsmi.bfs_submit(s, ids[k], r) for k, r in jobs]
        left, end = set(ts), time.time() + 30
        while left and time.time() < end:
            left -= set(bfsmi.bfs_server_completed(s))
            time.sleep(1e-4)
        assert not left
        for t, (k, r) in zip(ts, jobs):
            got = np.empty(gs[k].V, dtype=np.int32)
            assert bfsmi.bfs_poll(s, t, got)[0] == bfsmi.BFS_OK
            assert np.array_equal(got, oracle.bfs(gs[k].off, gs[k].col, r).level), (k, r)
    assert bfsmi.bfs_server_get_stats(s).failed == 0
    bfsmi.bfs_server_destroy(s)
    for h in hs:
        h.close()


@pytest.mark.parametrize("name", ["rmat12", "hub50021", "grid90", "rmat16"])
@pytest.mark.parametrize("R,C", [(1, 1), (4, 1), (2, 4), (8, 8)])
def test_blocked(bfsmi, name, R, C):
    g = GRAPHS[name]() if name in GRAPHS else _rmat(16)
    A = bfsmi.Grid2D.from_csr(g.off, g.col, R, C)
    B = bfsmi.Grid2D.from_csr(g.off, g.col, R, C)
    _lower(bfsmi, "bfs_test_grid2d_pack_limit", A.handle)
    for mode in (0, 1, 2):
        print("case", name, R, C, mode, flush=True)
        items = []
        for r in _roots(g, 2):
            lv, pa, st = A.run(r, msg_mode=mode)
            _, _, sb = B.run(r, msg_mode=mode)
            torch.cuda.synchronize()
            items.append((r, lv.cpu().numpy(), pa.cpu().numpy(), st))
            for f, _ in st._fields_:
                assert f == "device_ms" or getattr(st, f) == getattr(sb, f), (f, r)
        assert_parity(g, items, directed=name.startswith("hub"),
                      label="%s wide %dx%d mode %d" % (name, R, C, mode))
    A.close()
    B.close()
