"""Rows of 8-node brick meshes gathered from element records: any valence, both numberings,
constrained DOFs, the two sides of each dispatch line, chunks of elements, streams and capture."""
import sys
import threading

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import TOL, rowscaled_error, vec_error

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FORMS = [("mass", O.MASS), ("poisson", O.POISSON), ("elasticity", O.ELASTICITY), ("flow", O.NS_SUPG)]
PARAMS = {O.MASS: {"coef": 1.7}, O.POISSON: {"coef": 1.3}, O.ELASTICITY: {"coef": 2.0, "nu": 0.3},
          O.NS_SUPG: {"rho": 1.1, "mu": 0.02, "tau_m": 3e-3, "tau_c": 1e-2}}


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def cuda(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def fan_mesh(sectors, layers):
    """Quadrilaterals around one axis, extruded: an axis node has up to 2 * sectors elements;
    the last node belongs to no element."""
    t = np.pi * np.arange(2 * sectors) / sectors
    r = np.where(np.arange(2 * sectors) % 2 == 0, 1.0, 1.2)
    xy = np.concatenate([np.zeros((2, 1)), np.stack([r * np.cos(t), r * np.sin(t)])], axis=1)
    m = xy.shape[1]
    coords = np.concatenate([np.concatenate([xy, np.full((1, m), 0.4 * k)]) for k in range(layers + 1)], axis=1)
    coords = np.concatenate([coords, np.full((3, 1), 2.0)], axis=1)
    q = [(0, 1 + 2 * i, 1 + (2 * i + 2) % (2 * sectors), 2 + 2 * i) for i in range(sectors)]
    conn = [[a + m * (k + z) for z in (0, 1) for a in e] for k in range(layers) for e in q]
    return W.Mesh(coords, np.array(conn, np.int32).T.copy())


MESHES = [("one", lambda: W.permute_mesh(W.structured_mesh((1, 1, 1), jitter=0.1, seed=1), 2)[0]),
          ("perm", lambda: W.permute_mesh(W.structured_mesh((5, 4, 3), jitter=0.2, seed=3), 4)[0]),
          ("fan12", lambda: fan_mesh(12, 3)), ("fan3", lambda: fan_mesh(3, 1))]


def inputs(kind, mesh, prec, seed=5):
    nf = O.form_nf(kind, 3)
    dt = np.float64 if prec == 0 else np.float32
    ep = None if kind == O.NS_SUPG else W.lognormal_elem(mesh.n_elems, 0.4, seed).astype(dt)
    src = None if kind == O.NS_SUPG else W.uniform_nodal(nf, mesh.n_nodes, -1, 1, seed + 1).astype(dt)
    st = W.uniform_nodal(4, mesh.n_nodes, -1, 1, seed + 2).astype(dt) if kind == O.NS_SUPG else None
    return nf, ep, src, st


def assemble(mf, pat, kind, mesh, prec, ep, src, st, mask=None, **kw):
    return pat.assemble(mf.Form(kind, **PARAMS[kind]), cuda(mesh.coords), precision=prec, elem_param=cuda(ep),
                        nodal_src=cuda(src), lin_state=cuda(st), dirichlet=cuda(mask), **kw)


@pytest.mark.parametrize("masked", [False, True], ids=["free", "dirichlet"])
@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind", [f[1] for f in FORMS], ids=[f[0] for f in FORMS])
@pytest.mark.parametrize("make", [m[1] for m in MESHES], ids=[m[0] for m in MESHES])
def test_rows_match_oracle(mf, make, kind, numbering, prec, masked):
    mesh = make()
    nf, ep, src, st = inputs(kind, mesh, prec)
    say("rows", mesh.n_elems, "kind", kind, "numbering", numbering, "prec", prec, "masked", masked)
    opat = O.Pattern(mesh, nf, numbering=numbering)
    mask = None
    if masked:  # DOFs of nodes that belong to an element
        node = np.arange(mesh.n_nodes)[:, None] + mesh.n_nodes * np.arange(nf)[None] if numbering else \
            nf * np.arange(mesh.n_nodes)[:, None] + np.arange(nf)[None]
        mask = np.zeros(nf * mesh.n_nodes, np.uint8)
        mask[node[np.unique(mesh.conn)]] = np.random.default_rng(6).random((np.unique(mesh.conn).size, nf)) < 0.2
    up = lambda a: None if a is None else a.astype(np.float64)
    Kr, dr = O.assemble(opat, kind, PARAMS[kind], elem_param=up(ep), nodal_src=up(src), state=up(st), dirichlet=mask)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf, numbering=numbering)
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    assert pat.status()[0] == mf.OK
    assert rowscaled_error(opat, K.cpu().numpy(), Kr) <= TOL[prec]
    assert vec_error(d.cpu().numpy(), dr) <= TOL[prec]


def rowscaled_gpu(pat, K, Kref):
    rp = torch.from_numpy(pat.arrays()[0]).cuda().long()
    n = rp.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    amax = lambda v: torch.zeros(n, dtype=v.dtype, device="cuda").scatter_reduce_(0, row, v.abs(), "amax")
    return float((amax(K - Kref) / amax(Kref).clamp_min(1e-300 if K.dtype == torch.float64 else 1e-37)).max())


# both sides of each line between the grid kernel and the rows, the last sizes of one and the
# first of the other, and between rows with the geometry and element blocks; nodes above and below the 30000 of the eight-nodes-per-wave gather; element
# records that go in two chunks; planes above and below 1 MB of records
SIDES = [(O.NS_SUPG, 1, (21, 21, 22)), (O.NS_SUPG, 1, (22, 22, 21)), (O.NS_SUPG, 0, (3, 2, 4)),
         (O.ELASTICITY, 0, (27, 27, 27)), (O.ELASTICITY, 0, (28, 27, 27)), (O.POISSON, 0, (27, 27, 27)),
         (O.POISSON, 0, (28, 27, 27)), (O.MASS, 0, (32, 32, 30)), (O.POISSON, 1, (37, 37, 36)),
         (O.POISSON, 1, (37, 37, 37)), (O.POISSON, 0, (124, 123, 125)), (O.NS_SUPG, 1, (90, 88, 89)),
         (O.ELASTICITY, 0, (38, 37, 15)), (O.NS_SUPG, 0, (40, 39, 1)), (O.NS_SUPG, 0, (25, 23, 9)),
         (O.POISSON, 0, (41, 41, 41)), (O.POISSON, 0, (42, 41, 41)), (O.POISSON, 1, (42, 41, 41)),
         (O.MASS, 0, (53, 53, 53)), (O.MASS, 0, (54, 53, 53)), (O.MASS, 1, (54, 53, 53)),
         (O.ELASTICITY, 0, (23, 23, 23)), (O.ELASTICITY, 0, (24, 23, 24)), (O.ELASTICITY, 1, (35, 35, 36)),
         (O.ELASTICITY, 1, (36, 36, 35)), (O.ELASTICITY, 1, (62, 66, 61))]


@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind,prec,n", SIDES)
def test_rows_agree_with_scatter(mf, kind, prec, n, numbering):
    say("rows against scatter", kind, prec, n, numbering)
    mesh = W.structured_mesh(n, jitter=0.1, seed=2)
    nf, ep, src, st = inputs(kind, mesh, prec)
    mask = (np.random.default_rng(8).random(nf * mesh.n_nodes) < 0.02).astype(np.uint8)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf, numbering=numbering)
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    Kr, dr = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask, scatter=1)
    # each side is within TOL of the exact rows
    assert rowscaled_gpu(pat, K, Kr) <= 2 * TOL[prec]
    assert float((d - dr).abs().max() / dr.abs().max()) <= 2 * TOL[prec]


@pytest.mark.parametrize("masked", [False, True], ids=["free", "dirichlet"])
@pytest.mark.parametrize("prec", [0, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind,n", [(O.ELASTICITY, (22, 21, 20)), (O.NS_SUPG, (22, 21, 20)), (O.POISSON, (22, 21, 20)),
                                    (O.POISSON, (29, 28, 27)), (O.MASS, (29, 28, 27))])
def test_scattered_numbering(mf, kind, n, numbering, prec, masked):
    """Random numbering of enough elements for records by elements, against the scatter."""
    say("scattered", kind, n, numbering, prec, masked)
    mesh = W.permute_mesh(W.structured_mesh(n, jitter=0.2, seed=3), 4)[0]
    first = mesh.n_elems * np.ones(mesh.n_nodes, np.int64)  # each node's first element
    np.minimum.at(first, mesh.conn.ravel(), np.tile(np.arange(mesh.n_elems), 8))
    assert (np.abs(np.diff(first)) > 1024).sum() > mesh.n_nodes // 4
    nf, ep, src, st = inputs(kind, mesh, prec)
    mask = (np.random.default_rng(8).random(nf * mesh.n_nodes) < 0.02).astype(np.uint8) if masked else None
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf, numbering=numbering)
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    Kr, dr = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask, scatter=1)
    # each side is within TOL of the exact rows
    assert rowscaled_gpu(pat, K, Kr) <= 2 * TOL[prec]
    assert float((d - dr).abs().max() / dr.abs().max()) <= 2 * TOL[prec]


def test_calls_on_two_streams_and_threads(mf):
    say("two threads, a stream each, one pattern")
    mesh = W.permute_mesh(W.structured_mesh((14, 13, 12), jitter=0.2, seed=3), 4)[0]
    nf, ep, src, _ = inputs(O.ELASTICITY, mesh, 0)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf)
    form, coords = mf.Form(O.ELASTICITY, **PARAMS[O.ELASTICITY]), cuda(mesh.coords)
    eps = [cuda(ep * (1 + k)) for k in range(2)]
    want = [pat.assemble(form, coords, elem_param=e) for e in eps]
    got = [[], []]
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got[k].append(pat.assemble(form, coords, elem_param=eps[k]))
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for k in range(2):
        assert len(got[k]) == 20
        assert all(torch.equal(K, want[k][0]) and torch.equal(d, want[k][1]) for K, d in got[k])


@pytest.mark.parametrize("warm", [True, False])
def test_captured_calls(mf, warm):
    """Calls captured on one pattern: each replay gives the eager result, also with eager calls
    on the same pattern between the replays, and past the captures that have a workspace."""
    say("captured rows, warm", warm)
    mesh = W.permute_mesh(W.structured_mesh((6, 5, 4), jitter=0.2, seed=3), 4)[0]
    nf, ep, src, _ = inputs(O.ELASTICITY, mesh, 0)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf)
    form, coords = mf.Form(O.ELASTICITY, **PARAMS[O.ELASTICITY]), cuda(mesh.coords)
    K = torch.empty(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.empty(pat.n_rows, dtype=torch.float64, device="cuda")
    e, other, f = cuda(ep), cuda(2 * ep), cuda(src)
    if warm:
        pat.assemble(form, coords, elem_param=e, nodal_src=f)
    torch.cuda.synchronize()
    graphs = []
    for _ in range(10):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            pat.assemble(form, coords, elem_param=e, nodal_src=f, K=K, d=d)
        graphs.append(g)
    Kr, dr = pat.assemble(form, coords, elem_param=e, nodal_src=f)
    for k in (0, 9, 7, 0, 9, 8, 0):
        pat.assemble(form, coords, elem_param=other)
        K.fill_(-1.0)
        d.fill_(-1.0)
        graphs[k].replay()
        torch.cuda.synchronize()
        assert float((K - Kr).abs().max() / Kr.abs().max()) <= TOL[0], k
        assert float((d - dr).abs().max() / dr.abs().max()) <= TOL[0], k
