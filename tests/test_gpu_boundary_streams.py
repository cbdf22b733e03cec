"""Boundary forms of one pattern on several streams, threads and captures: every call's faces stay
its own."""
import sys
import threading

import numpy as np
import pytest

import oracle as O
import oracle.boundary as OB
import workloads as W
from helpers import TOL

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

VALUE = [0.0, 0.0, 0.0, 1.0, 0.05]


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def flow_case(mf, n=(9, 8, 7)):
    mesh = W.structured_mesh(n, jitter=0.15, seed=2)
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, 4)
    sets = [tuple(cuda(a) for a in W.box_faces(n, sides=s)) for s in ([0, 2, 4], [1, 3, 5])]
    return pat, cuda(mesh.coords), cuda(W.uniform_nodal(4, mesh.n_nodes, -1, 1, 3)), sets


def test_flow_forms_on_two_streams_and_threads(mf):
    """Two threads with a stream and a face set each; the forms' sums do not depend on the run."""
    say("flow boundary forms, two threads, a stream each, one pattern")
    pat, coords, state, sets = flow_case(mf)
    call = lambda s: pat.assemble_boundary(OB.NS_OUTFLOW, coords, *s, coef=2.0, value=VALUE, state=state)  # noqa: E731
    want = [call(s) for s in sets]
    got = [[], []]
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got[k].append(call(sets[k]))
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for k in range(2):
        assert len(got[k]) == 20
        assert all(torch.equal(K, want[k][0]) and torch.equal(d, want[k][1]) for K, d in got[k])


def test_captured_flow_forms(mf):
    """Ten captures, two of them past those that have a workspace of their own: each replay adds its
    own faces, with an eager call of the other faces between."""
    say("captured flow boundary forms")
    pat, coords, state, sets = flow_case(mf, (5, 4, 3))
    kw = dict(coef=2.0, value=VALUE, state=state)
    K = torch.zeros(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.zeros(pat.n_rows, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graphs = []
    for k in range(10):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            pat.assemble_boundary(OB.NS_OUTFLOW, coords, *sets[k % 2], K=K, d=d, **kw)
        graphs.append(g)
    want = [pat.assemble_boundary(OB.NS_OUTFLOW, coords, *s, **kw) for s in sets]
    for k in (0, 9, 8, 1, 9, 0, 8):
        pat.assemble_boundary(OB.NS_OUTFLOW, coords, *sets[1 - k % 2], **kw)
        K.zero_()
        d.zero_()
        graphs[k].replay()
        torch.cuda.synchronize()
        assert torch.equal(K, want[k % 2][0]) and torch.equal(d, want[k % 2][1]), k


@pytest.mark.parametrize("elem", ["tet10", "quad8"])
def test_ninth_capture(mf, elem):
    """Assembly and then faces enough for a larger workspace, in eight captures; a ninth refuses the
    boundary form, names the captures as the reason and stays a capture."""
    say("nine captures", elem)
    mesh = W.tet10_mesh((2, 2, 2), jitter=0.1, seed=2) if elem == "tet10" else W.serendipity_mesh_2d((6, 5), jitter=0.1, seed=2)
    keys = np.arange(4 * mesh.n_elems)
    fe, fi = cuda((keys // 4).astype(np.int32)), cuda((keys % 4).astype(np.uint8))
    pat, coords = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, mesh.dim, 1), cuda(mesh.coords)
    form = mf.Form(O.POISSON, coef=1.3)
    K = torch.empty(pat.nnz, dtype=torch.float64, device="cuda")
    d = torch.empty(pat.n_rows, dtype=torch.float64, device="cuda")

    def system(K, d):
        pat.assemble(form, coords, K=K, d=d)
        pat.assemble_boundary(OB.CONVECTION, coords, fe, fi, coef=2.0, value=[0.3], K=K, d=d)

    torch.cuda.synchronize()
    graphs = [torch.cuda.CUDAGraph() for _ in range(9)]
    for g in graphs[:8]:
        with torch.cuda.graph(g):
            system(K, d)
    with torch.cuda.graph(graphs[8]):
        pat.assemble(form, coords, K=K, d=d)
        with pytest.raises(mf.MFError, match="8 captures") as err:
            pat.assemble_boundary(OB.CONVECTION, coords, fe, fi, coef=2.0, value=[0.3], K=K, d=d)
    assert err.value.status == mf.ERR_UNSUPPORTED
    Kr, dr = torch.empty_like(K), torch.empty_like(d)
    system(Kr, dr)
    Kd, dd = pat.assemble(form, coords)
    for k in (0, 8, 7, 0, 8, 3):
        system(Kd.clone(), dd.clone())
        K.fill_(-1.0)
        d.fill_(-1.0)
        graphs[k].replay()
        torch.cuda.synchronize()
        a, b = (Kd, dd) if k == 8 else (Kr, dr)
        assert float((K - a).abs().max()) <= TOL[0] * float(a.abs().max()), k
        assert float((d - b).abs().max()) <= TOL[0] * float(dr.abs().max()), k
