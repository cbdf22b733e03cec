"""The arrays of a pattern, which share their allocations: node counts on both sides of the scan's tiles
and levels, against the grid's rows, with another pattern made and destroyed meanwhile."""
import ctypes as C
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def grid_rows(nx, ny):
    """row_ptr and col_idx of scalar rows on a grid of nx x ny quadrilaterals."""
    i, j = np.meshgrid(np.arange(nx + 1), np.arange(ny + 1), indexing="xy")
    cols = np.stack([np.where((i + a >= 0) & (i + a <= nx) & (j + b >= 0) & (j + b <= ny),
                              (i + a) + (nx + 1) * (j + b), -1).ravel()
                     for b in (-1, 0, 1) for a in (-1, 0, 1)], 1)
    return np.concatenate([[0], np.cumsum((cols >= 0).sum(1))]), cols[cols >= 0]


# nodes: 4, 1023, 1024 and 1025 (tiles of 1024 counts), 1024^2 and more (two levels of tiles)
@pytest.mark.parametrize("n", [(1, 1), (92, 10), (31, 31), (40, 24), (1023, 1023), (1023, 1024)])
def test_arrays(mf, n):
    print("[case] pattern arrays", n, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n)
    conn = torch.from_numpy(mesh.conn).cuda()
    mf.Pattern(conn, mesh.n_nodes, 2, 2)
    pat = mf.Pattern(conn, mesh.n_nodes, 2, 1)
    other = mf.Pattern(conn, mesh.n_nodes, 2, 3)
    rp, ci, rank = pat.arrays()
    rows, cols = grid_rows(*n)
    assert np.array_equal(rp, rows) and np.array_equal(ci, cols)
    a, b = np.divmod(np.arange(16), 4)
    at = rows[mesh.conn[a]] + rank.reshape(16, -1)
    assert np.array_equal(cols[at], mesh.conn[b])
    p = [C.c_void_p() for _ in range(3)]
    lib = mf.load()
    lib.mf_pattern_info(pat.handle, None, None, *[C.byref(q) for q in p])
    assert all(q.value % 256 == 0 for q in p)
    del other


def test_bad_mesh_then_good(mf):
    print("[case] pattern of a bad mesh, then a good one", file=sys.stderr, flush=True)
    mesh = W.structured_mesh((40, 24))
    bad = mesh.conn.copy()
    bad[2, 17] = mesh.n_nodes
    for _ in range(3):
        with pytest.raises(mf.MFError) as e:
            mf.Pattern(torch.from_numpy(bad).cuda(), mesh.n_nodes, 2, 1)
        assert e.value.status == mf.ERR_BAD_MESH
    rp, ci, _ = mf.Pattern(torch.from_numpy(mesh.conn).cuda(), mesh.n_nodes, 2, 1).arrays()
    rows, cols = grid_rows(40, 24)
    assert np.array_equal(rp, rows) and np.array_equal(ci, cols)
