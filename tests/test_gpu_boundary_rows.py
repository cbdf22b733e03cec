"""Boundary forms gathered node by node: faces listed several times and in any order, every face
of an element, faces per call on both sides of a workgroup, and captured calls."""
import sys

import numpy as np
import pytest

import oracle as O
import oracle.boundary as OB
import oracle.serendipity as S
import workloads as W
from helpers import TOL, rowscaled_sparse

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ELEMS = {"hex8": (lambda: W.structured_mesh((3, 2, 2), jitter=0.15, seed=2), 6, O.Pattern, OB.assemble_boundary),
         "hex20": (lambda: W.serendipity_mesh((2, 1, 2), jitter=0.1, seed=2), 6, S.Pattern20, S.assemble_boundary20),
         "tet10": (lambda: W.tet10_mesh((1, 1, 2), jitter=0.1, seed=2), 4, S.Pattern20, S.assemble_boundary_tet10),
         "quad4": (lambda: W.structured_mesh((4, 3), jitter=0.15, seed=2), 4, O.Pattern, OB.assemble_boundary_2d),
         "quad8": (lambda: W.serendipity_mesh_2d((4, 3), jitter=0.1, seed=2), 4, S.Pattern20, OB.assemble_boundary_2d)}


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def case(elem, n_faces):
    mesh = ELEMS[elem][0]()
    rng = np.random.default_rng(n_faces)
    fe = rng.integers(0, mesh.n_elems, n_faces).astype(np.int32)  # interior faces and repeats included
    fi = rng.integers(0, ELEMS[elem][1], n_faces).astype(np.uint8)
    k = min(n_faces, ELEMS[elem][1])
    fe[:k], fi[:k] = mesh.n_elems - 1, np.arange(k)  # every face of one element
    return mesh, fe, fi


@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("vector", [False, True])
@pytest.mark.parametrize("n_faces", [1, 5, 300])
@pytest.mark.parametrize("elem", list(ELEMS))
def test_repeated_faces(mf, elem, n_faces, vector, numbering, prec):
    mesh, fe, fi = case(elem, n_faces)
    nf = mesh.dim if vector else 1
    say("repeated faces", elem, n_faces, "nf", nf, "numbering", numbering, "prec", prec)
    dt = np.float64 if prec == 0 else np.float32
    state = W.uniform_nodal(nf, mesh.n_nodes, 0.5, 1.5, 3).astype(dt)
    value = [0.1, -0.2, 0.3][:nf]
    opat = ELEMS[elem][2](mesh, nf, numbering=numbering)
    Kr, dr = ELEMS[elem][3](opat, OB.PENALTY, 3.0, value, fe, fi, state=state.astype(np.float64))
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, mesh.dim, nf, numbering=numbering)
    K, d = pat.assemble_boundary(OB.PENALTY, cuda(mesh.coords), cuda(fe), cuda(fi), coef=3.0, value=value,
                                 state=cuda(state), precision=prec)
    assert pat.status()[0] == mf.OK
    import scipy.sparse as sp
    Kg = sp.csr_matrix((K.double().cpu().numpy(), opat.col_idx, opat.row_ptr), shape=(opat.n_rows, opat.n_rows))
    assert rowscaled_sparse(Kg, sp.csr_matrix(Kr)) <= TOL[prec]
    assert np.abs(d.double().cpu().numpy() - dr).max() <= TOL[prec] * np.abs(dr).max()


@pytest.mark.parametrize("elem", list(ELEMS))
def test_captured_boundary(mf, elem):
    """The form adds into K and d, so a replay adds the same once more."""
    say("captured boundary", elem)
    mesh, fe, fi = case(elem, 20)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, mesh.dim, 1)
    coords, fe, fi = cuda(mesh.coords), cuda(fe), cuda(fi)
    state = cuda(W.uniform_nodal(1, mesh.n_nodes, 0.5, 1.5, 3))
    K = torch.zeros(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.zeros(pat.n_rows, dtype=torch.float64, device="cuda")
    kw = dict(coef=2.0, value=[0.3], state=state)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        pat.assemble_boundary(OB.PENALTY, coords, fe, fi, K=K, d=d, **kw)
    Kr, dr = pat.assemble_boundary(OB.PENALTY, coords, fe, fi, **kw)
    for k in range(1, 4):
        g.replay()
        pat.assemble_boundary(OB.PENALTY, coords, fe[:3], fi[:3], **kw)
        torch.cuda.synchronize()
        assert float((K - k * Kr).abs().max()) <= TOL[0] * float(Kr.abs().max()) * k
        assert float((d - k * dr).abs().max()) <= TOL[0] * float(dr.abs().max()) * k
