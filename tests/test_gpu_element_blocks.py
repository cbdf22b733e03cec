"""Element blocks of the quadratic elements and their gather into rows: remainders of a wave's
elements, constrained DOFs, element chunks and captured calls."""
import sys

import numpy as np
import pytest

import oracle as O
import oracle.serendipity as S
import workloads as W
from helpers import TOL, rowscaled_sparse, submesh_for_nodes

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PARAMS = {O.MASS: {"coef": 1.7}, O.POISSON: {"coef": 1.3}, O.ELASTICITY: {"coef": 2.0, "nu": 0.3},
          O.NS_SUPG: {"rho": 1.1, "mu": 0.02, "tau_m": 3e-3, "tau_c": 1e-2}}
MAKE = {"hex20": W.serendipity_mesh, "tet10": W.tet10_mesh, "quad8": W.serendipity_mesh_2d}


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def cuda(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def fields(kind, mesh):
    return {O.MASS: 1, O.POISSON: 1, O.ELASTICITY: mesh.dim, O.NS_SUPG: mesh.dim + 1}[kind]


def inputs(kind, mesh, prec):
    nf, dt = fields(kind, mesh), np.float64 if prec == 0 else np.float32
    if kind == O.NS_SUPG:
        return nf, None, None, W.uniform_nodal(nf, mesh.n_nodes, -1, 1, 7).astype(dt)
    return nf, W.lognormal_elem(mesh.n_elems, 0.4, 5).astype(dt), W.uniform_nodal(nf, mesh.n_nodes, -1, 1, 6).astype(dt), None


def assemble(mf, pat, kind, mesh, prec, ep, src, st, mask=None, **kw):
    return pat.assemble(mf.Form(kind, **PARAMS[kind]), cuda(mesh.coords), precision=prec, elem_param=cuda(ep),
                        nodal_src=cuda(src), lin_state=cuda(st), dirichlet=cuda(mask), **kw)


@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind", [O.MASS, O.POISSON, O.ELASTICITY, O.NS_SUPG])
@pytest.mark.parametrize("elem,n", [("hex20", (1, 1, 1)), ("hex20", (3, 1, 2)), ("tet10", (1, 1, 1)), ("tet10", (1, 2, 2)),
                                    ("quad8", (1, 1)), ("quad8", (5, 3))])
def test_blocks_with_constrained_dofs(mf, elem, n, kind, numbering, prec):
    mesh = MAKE[elem](n, jitter=0.15, seed=2)
    say("blocks", elem, n, "kind", kind, "numbering", numbering, "prec", prec)
    nf, ep, src, st = inputs(kind, mesh, prec)
    opat = S.Pattern20(mesh, nf, numbering)
    up = lambda a: None if a is None else a.astype(np.float64)
    Kr, dr = S.assemble20(opat, kind, PARAMS[kind], elem_param=up(ep), nodal_src=up(src), state=up(st))
    mask = (np.random.default_rng(3).random(opat.n_rows) < 0.15).astype(np.uint8)
    row = np.repeat(np.arange(opat.n_rows), np.diff(opat.row_ptr))
    Kr = np.where(mask[row] | mask[opat.col_idx], (row == opat.col_idx).astype(np.float64), np.asarray(Kr))
    dr = np.where(mask, 0.0, dr)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, mesh.dim, nf, numbering=numbering)
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    assert pat.status()[0] == mf.OK
    import scipy.sparse as sp
    csr = lambda v: sp.csr_matrix((v, opat.col_idx, opat.row_ptr), shape=(opat.n_rows, opat.n_rows))
    assert rowscaled_sparse(csr(K.double().cpu().numpy()), csr(Kr)) <= TOL[prec]
    assert np.abs(d.double().cpu().numpy() - dr).max() <= TOL[prec] * np.abs(dr).max()


def test_blocks_in_chunks(mf):
    """More element blocks than the workspace holds at once: rows on both sides of the cut."""
    say("hex20 elasticity f32 in chunks")
    mesh = W.serendipity_mesh((43, 42, 41), jitter=0.1, seed=2)
    nf, ep, src, _ = inputs(O.ELASTICITY, mesh, 1)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf)
    K, d = assemble(mf, pat, O.ELASTICITY, mesh, 1, ep, src, None)
    rp = pat.arrays()[0]
    cut = (1 << 30) // (4 * 60 * 61 + 1)
    assert cut < mesh.n_elems
    nodes = np.unique(np.concatenate([mesh.conn[[0, 7, 9], cut - 1], mesh.conn[[0, 19], cut], mesh.conn[[7], -1], [0]]))
    sub, elems, used, local = submesh_for_nodes(mesh, nodes)
    opat = S.Pattern20(sub, nf)
    Kr, dr = S.assemble20(opat, O.ELASTICITY, PARAMS[O.ELASTICITY], elem_param=ep[elems].astype(np.float64),
                          nodal_src=src[:, used].astype(np.float64))
    for v in nodes:
        for i in range(nf):
            a, r = int(rp[nf * v + i]), nf * local[v] + i
            b = slice(opat.row_ptr[r], opat.row_ptr[r + 1])
            got = K[a:int(rp[nf * v + i + 1])].double().cpu().numpy()
            assert np.abs(got - Kr[b]).max() <= TOL[1] * np.abs(Kr[b]).max()
            assert abs(float(d[nf * v + i]) - dr[r]) <= TOL[1] * np.abs(dr).max()


@pytest.mark.parametrize("kind", [O.POISSON, O.ELASTICITY, O.NS_SUPG])
@pytest.mark.parametrize("elem", ["hex20", "tet10", "quad8"])
def test_captured_blocks(mf, elem, kind):
    say("captured blocks", elem, kind)
    mesh = MAKE[elem]((3, 2) if elem == "quad8" else (3, 2, 2), jitter=0.15, seed=2)
    nf, ep, src, st = inputs(kind, mesh, 0)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, mesh.dim, nf)
    form, coords = mf.Form(kind, **PARAMS[kind]), cuda(mesh.coords)
    args = dict(elem_param=cuda(ep), nodal_src=cuda(src), lin_state=cuda(st))
    K = torch.empty(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.empty(pat.n_rows, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graphs = []
    for _ in range(9):  # the last has no workspace of its own
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            pat.assemble(form, coords, K=K, d=d, **args)
        graphs.append(g)
    Kr, dr = pat.assemble(form, coords, **args)
    for k in (0, 8, 3, 0, 8):
        pat.assemble(form, 2.0 * coords, **args)
        K.fill_(-1.0)
        d.fill_(-1.0)
        graphs[k].replay()
        torch.cuda.synchronize()
        assert float((K - Kr).abs().max()) <= TOL[0] * float(Kr.abs().max())
        assert float((d - dr).abs().max()) <= TOL[0] * float(dr.abs().max())
