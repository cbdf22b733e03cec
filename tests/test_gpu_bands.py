"""Bands of grid planes with any remainder: planes and workgroups of 16 and 32 nodes that divide in no way, few
and many planes, constrained DOFs in single elements, against the independent scatter."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import TOL
from test_gpu_rows import assemble, cuda, inputs, rowscaled_gpu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# flow planes of 1850 B and elasticity planes of 770 B an element that hold more than 2.5 MB
PLANES = [(O.NS_SUPG, (37, 37, 3)), (O.NS_SUPG, (1400, 1, 1)), (O.NS_SUPG, (53, 29, 2)), (O.NS_SUPG, (38, 40, 7)),
          (O.ELASTICITY, (61, 59, 5)), (O.ELASTICITY, (1, 3300, 4)), (O.ELASTICITY, (73, 47, 4))]


@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("kind,n", PLANES)
def test_planes(mf, kind, n, numbering):
    print("[case] bands", kind, n, numbering, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n, jitter=0.1, seed=2)
    nf, ep, src, st = inputs(kind, mesh, 0)
    mask = np.zeros(nf * mesh.n_nodes, np.uint8)
    mask[np.random.default_rng(8).integers(0, mask.size, 9)] = 1
    mask[[0, -1]] = 1
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf, numbering=numbering)
    assert pat.grid()[0]
    K, d = assemble(mf, pat, kind, mesh, 0, ep, src, st, mask)
    assert pat.status()[0] == mf.OK
    Kr, dr = assemble(mf, pat, kind, mesh, 0, ep, src, st, mask, scatter=1)
    # each side is within TOL of the exact rows
    assert rowscaled_gpu(pat, K, Kr) <= 2 * TOL[0]
    assert float((d - dr).abs().max() / dr.abs().max()) <= 2 * TOL[0]
