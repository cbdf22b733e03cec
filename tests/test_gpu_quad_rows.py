"""Rows of 4-node quadrilateral meshes: any valence (up to a hub whose rows do not fit the LDS, which
goes colour by colour), both numberings, constrained DOFs, row counts around a wave, capture."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import TOL, rowscaled_error, vec_error

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PARAMS = {O.MASS: {"coef": 1.7}, O.POISSON: {"coef": 1.3}, O.ELASTICITY: {"coef": 2.0, "nu": 0.3},
          O.NS_SUPG: {"rho": 1.1, "mu": 0.02, "tau_m": 3e-3, "tau_c": 1e-2}}


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def cuda(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def fan(sectors):
    """Quadrilaterals around one node; the last node belongs to no element."""
    t = np.pi * np.arange(2 * sectors) / sectors
    r = np.where(np.arange(2 * sectors) % 2 == 0, 1.0, 1.2)
    xy = np.concatenate([np.zeros((2, 1)), np.stack([r * np.cos(t), r * np.sin(t)]), np.full((2, 1), 3.0)], axis=1)
    q = [(0, 1 + 2 * i, 1 + (2 * i + 2) % (2 * sectors), 2 + 2 * i) for i in range(sectors)]
    return W.Mesh(xy, np.array(q, np.int32).T.copy())


MESHES = [("one", lambda: W.structured_mesh((1, 1), jitter=0.1, seed=1)),
          ("5x3", lambda: W.structured_mesh((5, 3), jitter=0.2, seed=1)),
          ("perm", lambda: W.permute_mesh(W.structured_mesh((7, 8), jitter=0.2, seed=3), 4)[0]),
          ("fan3", lambda: fan(3)), ("fan9", lambda: fan(9)), ("fan85", lambda: fan(85)), ("fan100", lambda: fan(100))]


@pytest.mark.parametrize("masked", [False, True], ids=["free", "dirichlet"])
@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind", list(PARAMS))
@pytest.mark.parametrize("make", [m[1] for m in MESHES], ids=[m[0] for m in MESHES])
def test_rows_match_oracle(mf, make, kind, numbering, prec, masked):
    mesh = make()
    nf = O.form_nf(kind, 2)
    say("quad rows", mesh.n_elems, "kind", kind, "numbering", numbering, "prec", prec, "masked", masked)
    dt = np.float64 if prec == 0 else np.float32
    flow = kind == O.NS_SUPG
    ep = None if flow else W.lognormal_elem(mesh.n_elems, 0.4, 5).astype(dt)
    src = None if flow else W.uniform_nodal(nf, mesh.n_nodes, -1, 1, 6).astype(dt)
    st = W.uniform_nodal(3, mesh.n_nodes, -1, 1, 7).astype(dt) if flow else None
    opat = O.Pattern(mesh, nf, numbering=numbering)
    mask = None
    if masked:  # DOFs of nodes that belong to an element
        node = np.arange(mesh.n_nodes)[:, None] + mesh.n_nodes * np.arange(nf)[None] if numbering else \
            nf * np.arange(mesh.n_nodes)[:, None] + np.arange(nf)[None]
        used = np.unique(mesh.conn)
        mask = np.zeros(nf * mesh.n_nodes, np.uint8)
        mask[node[used]] = np.random.default_rng(6).random((used.size, nf)) < 0.2
    up = lambda a: None if a is None else a.astype(np.float64)
    Kr, dr = O.assemble(opat, kind, PARAMS[kind], elem_param=up(ep), nodal_src=up(src), state=up(st), dirichlet=mask)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 2, nf, numbering=numbering)
    K, d = pat.assemble(mf.Form(kind, **PARAMS[kind]), cuda(mesh.coords), precision=prec, elem_param=cuda(ep),
                        nodal_src=cuda(src), lin_state=cuda(st), dirichlet=cuda(mask))
    assert pat.status()[0] == mf.OK
    assert rowscaled_error(opat, K.cpu().numpy(), Kr) <= TOL[prec]
    assert vec_error(d.cpu().numpy(), dr) <= TOL[prec]


def test_captured_and_bad_element(mf):
    """A captured call on a pattern that was never assembled, and the report of an inverted
    element, which adds nothing and is cleared by the next call."""
    say("captured quads")
    mesh = W.structured_mesh((9, 7), jitter=0.2, seed=3)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 2, 1)
    coords, src = cuda(mesh.coords), cuda(W.uniform_nodal(1, mesh.n_nodes, -1, 1, 6))
    K = torch.empty(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.empty(pat.n_rows, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        pat.assemble(mf.Form(mf.POISSON), coords, nodal_src=src, K=K, d=d)
    Kr, dr = pat.assemble(mf.Form(mf.POISSON), coords, nodal_src=src)
    flipped = coords.clone()
    flipped[0, 0] = 5.0  # node 0 past its element's other side
    for _ in range(3):
        Kb, _ = pat.assemble(mf.Form(mf.POISSON), flipped, nodal_src=src)
        assert pat.status() == (mf.ERR_BAD_JACOBIAN, 0)
        assert float(Kb[0]) == 0.0
        K.fill_(-1.0)
        d.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(K, Kr) and torch.equal(d, dr) and pat.status()[0] == mf.OK
