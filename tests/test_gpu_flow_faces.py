"""Flow boundary forms by kind: several faces of an element, faces listed more than once, interior faces,
with and without a target, and degenerate faces and elements."""
import sys

import numpy as np
import pytest

import oracle as O
import oracle.boundary as OB
import workloads as W
from helpers import TOL, rowscaled_sparse

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

VALUE = [0.3, -0.2, 0.1, 1.2, 0.05]


def cuda(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("with_target", [False, True])
@pytest.mark.parametrize("kind", [OB.NS_INFLOW, OB.NS_OUTFLOW, OB.NS_FIX])
def test_repeated_flow_faces(mf, kind, with_target, numbering, prec):
    print("[case] flow faces", kind, with_target, numbering, prec, file=sys.stderr, flush=True)
    mesh = W.structured_mesh((3, 2, 2), jitter=0.15, seed=2)
    rng = np.random.default_rng(5)
    fe, fi = rng.integers(0, mesh.n_elems, 40).astype(np.int32), rng.integers(0, 6, 40).astype(np.uint8)
    fe[:6], fi[:6] = mesh.n_elems - 1, np.arange(6)
    dt = np.float64 if prec == 0 else np.float32
    state = W.uniform_nodal(4, mesh.n_nodes, -1, 1, 3).astype(dt)
    target = W.uniform_nodal(4, mesh.n_nodes, -1, 1, 4).astype(dt) if with_target else None
    up = lambda a: None if a is None else a.astype(np.float64)  # noqa: E731
    opat = O.Pattern(mesh, 4, numbering=numbering)
    Kr, dr = OB.assemble_boundary(opat, kind, 2.0, VALUE, fe, fi, state=up(state), target=up(target))
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, 4, numbering=numbering)
    K, d = pat.assemble_boundary(kind, cuda(mesh.coords), cuda(fe), cuda(fi), coef=2.0, value=VALUE, state=cuda(state),
                                 target=cuda(target), precision=prec)
    assert pat.status()[0] == mf.OK
    import scipy.sparse as sp
    Kg = sp.csr_matrix((K.double().cpu().numpy(), opat.col_idx, opat.row_ptr), shape=(opat.n_rows, opat.n_rows))
    assert rowscaled_sparse(Kg, sp.csr_matrix(Kr)) <= TOL[prec]
    assert np.abs(d.double().cpu().numpy() - dr).max() <= TOL[prec] * np.abs(dr).max()


@pytest.mark.parametrize("kind", [OB.NS_INFLOW, OB.NS_OUTFLOW, OB.NS_FIX])
@pytest.mark.parametrize("bad", ["face", "element"])
def test_degenerate(mf, kind, bad):
    """A face of no area, or one of an element turned inside out, is reported; its element adds nothing."""
    print("[case] degenerate flow face", kind, bad, file=sys.stderr, flush=True)
    mesh = W.structured_mesh((2, 1, 1))
    coords = mesh.coords.copy()
    right = mesh.conn[:, 1]
    if bad == "face":
        coords[:, right[[1, 3, 5, 7]]] = coords[:, right[[1]]]
    else:
        coords[0, right[[1, 3, 5, 7]]] = -1.0
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, 4)
    call = lambda e, f: pat.assemble_boundary(kind, cuda(coords), cuda(np.array(e, np.int32)), cuda(np.array(f, np.uint8)),  # noqa: E731
                                              coef=2.0, value=VALUE)
    K0, d0 = call([0], [0])
    assert pat.status()[0] == mf.OK
    K, d = call([0, 1], [0, 1])
    assert pat.status()[0] == mf.ERR_BAD_JACOBIAN and pat.status()[1] == 1
    assert torch.equal(K, K0) and torch.equal(d, d0)
