"""Eager calls whose workspace is made or grown while the same thread captures another stream: the
capture goes on, and both sides' results are the usual ones."""
import sys

import numpy as np
import pytest

import oracle as O
import oracle.boundary as OB
import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("mode", ["global", "thread_local"])
def test_eager_calls_during_a_capture(mf, mode):
    print("[case] eager calls beside a capture,", mode, file=sys.stderr, flush=True)
    mesh = W.permute_mesh(W.structured_mesh((6, 5, 4), jitter=0.2, seed=3), 4)[0]
    keys = np.arange(6 * mesh.n_elems)
    fe, fi = cuda((keys // 6).astype(np.int32)), cuda((keys % 6).astype(np.uint8))
    coords, form = cuda(mesh.coords), mf.Form(O.ELASTICITY, coef=2.0, nu=0.3)
    warm, cold = (mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, 3) for _ in range(2))
    K = torch.empty(cold.nnz, dtype=torch.float64, device="cuda")
    d = torch.empty(cold.n_rows, dtype=torch.float64, device="cuda")
    x = torch.zeros(64, device="cuda")

    def system(pat, K, d, stream=None):  # the faces' rows need a larger workspace than the elements
        pat.assemble(form, coords, K=K, d=d, stream=stream)
        pat.assemble_boundary(OB.PENALTY, coords, fe, fi, coef=3.0, K=K, d=d, stream=stream)

    Kr, dr = torch.empty_like(K), torch.empty_like(d)
    system(warm, Kr, dr)
    torch.cuda.synchronize()
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, capture_error_mode=mode):
        x.add_(1.0)
        system(cold, K, d, side)
        x.add_(1.0)
    side.synchronize()
    assert torch.equal(K, Kr) and torch.equal(d, dr)
    for k in range(1, 4):
        system(cold, K, d)
        g.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == 2.0 * k and torch.equal(K, Kr)
