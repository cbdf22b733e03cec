"""Small meshes of 4-node quadrilaterals on both sides of the lines of the one-workgroup call: one and two
passes of its waves over the rows, the last rows it takes and the first it does not."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import TOL, rowscaled_error, vec_error
from test_gpu_quad_rows import PARAMS, cuda

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# rows: 256 | 272, 384 | 400 of scalar forms; 64 | 66 of elasticity
CASES = [(k, n) for k in (O.MASS, O.POISSON) for n in ((15, 15), (16, 15), (23, 15), (24, 15))] + \
        [(O.ELASTICITY, n) for n in ((3, 7), (10, 2))]


@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("masked", [False, True], ids=["free", "dirichlet"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("kind,n", CASES)
def test_small_quads(mf, kind, n, shuffled, masked, prec):
    print("[case] small quads", kind, n, shuffled, masked, prec, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n, jitter=0.2, seed=1)
    if shuffled:
        mesh = W.permute_mesh(mesh, 4)[0]
    nf, dt = (2 if kind == O.ELASTICITY else 1), np.float64 if prec == 0 else np.float32
    ep = W.lognormal_elem(mesh.n_elems, 0.4, 5).astype(dt)
    src = W.uniform_nodal(nf, mesh.n_nodes, -1, 1, 6).astype(dt)
    mask = (np.random.default_rng(6).random(nf * mesh.n_nodes) < 0.2).astype(np.uint8) if masked else None
    opat = O.Pattern(mesh, nf)
    Kr, dr = O.assemble(opat, kind, PARAMS[kind], elem_param=ep.astype(np.float64), nodal_src=src.astype(np.float64),
                        dirichlet=mask)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 2, nf)
    call = lambda e: pat.assemble(mf.Form(kind, **PARAMS[kind]), cuda(mesh.coords), precision=prec, elem_param=cuda(e),  # noqa: E731
                                  nodal_src=cuda(src), dirichlet=cuda(mask))
    wrong = ep.copy()
    wrong[-1] = np.nan
    call(wrong)
    assert pat.status() == (mf.ERR_NONFINITE, mesh.n_elems - 1)
    K, d = call(ep)  # the status is the last call's
    assert pat.status()[0] == mf.OK
    assert rowscaled_error(opat, K.cpu().numpy(), Kr) <= TOL[prec]
    assert vec_error(d.cpu().numpy(), dr) <= TOL[prec]
