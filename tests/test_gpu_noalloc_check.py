"""The allocation-free search's CSR check, which the search's kernels read
themselves: a fault in the first or the last entries of one or many checking
workgroups stops the search before it writes anything, and the next call is
as if it had not been."""
import ctypes

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1408_1605_amd import binding
    binding.load()
    return binding


def _run(lib, off, col, root):
    V = len(off) - 1
    d_off, d_col = torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda()
    lv = torch.full((V,), -7, dtype=torch.int32, device="cuda")
    pa = torch.full((V,), -7, dtype=torch.int32, device="cuda")
    so = lib.load()
    st = so.bfs_run_noalloc.argtypes[-1]._type_()
    code = so.bfs_run_noalloc(V, len(col), d_off.data_ptr(), d_col.data_ptr(), root,
                              lv.data_ptr(), pa.data_ptr(),
                              torch.cuda.current_stream().cuda_stream, ctypes.byref(st))
    torch.cuda.synchronize()
    return code, lv.cpu().numpy(), pa.cpu().numpy()


# edges: fewer than vertices, one checking workgroup, many
@pytest.mark.parametrize("n,m", [(1, 0), (3_000, 200), (100, 900), (5_000, 60_000)])
def test_faults_then_a_valid_call(lib, n, m):
    rng = np.random.default_rng(n)
    g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m))
    off, col = np.ascontiguousarray(g.off, np.int64), np.ascontiguousarray(g.col, np.int32)
    print("case", n, m, flush=True)
    faults = []
    for v in (0, n):
        o = off.copy()
        o[v] += 1 if v else -1
        faults.append((o, col))
    if n > 2:
        o = off.copy()
        o[n - 1] = off[n] + 5
        faults.append((o, col))
    for e in (0, len(col) - 1) if len(col) else ():
        for bad in (-1, n):
            c = col.copy()
            c[e] = bad
            faults.append((off, c))
    for o, c in faults:
        code, lv, pa = _run(lib, o, c, n // 2)
        assert code == lib.BFS_ERR_INVALID
        assert (lv == -7).all() and (pa == -7).all()
        code, lv, pa = _run(lib, off, col, n // 2)
        assert code == lib.BFS_OK
        assert np.array_equal(lv, oracle.bfs(off, col, n // 2).level)
        assert oracle.validate(off, col, n // 2, lv, pa)[0] == 0
