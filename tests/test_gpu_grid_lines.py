"""Structured grids on both sides of each line between the column kernel and the rows, with and without
constrained DOFs, against the independent scatter."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import TOL
from test_gpu_rows import assemble, cuda, inputs, rowscaled_gpu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FREE, FIXED = False, True
# the last size of one kernel and the first of the other
LINES = [(O.POISSON, 0, FIXED, (15, 15, 15)), (O.POISSON, 0, FIXED, (16, 15, 15)), (O.MASS, 0, FIXED, (20, 20, 21)),
         (O.MASS, 0, FIXED, (20, 21, 21)), (O.POISSON, 1, FIXED, (22, 21, 21)), (O.POISSON, 1, FIXED, (22, 21, 22)),
         (O.MASS, 1, FIXED, (22, 21, 21)), (O.MASS, 1, FIXED, (22, 21, 22)), (O.POISSON, 1, FREE, (15, 15, 15)),
         (O.ELASTICITY, 0, FREE, (32, 32, 31)), (O.ELASTICITY, 0, FREE, (32, 32, 32)),
         (O.ELASTICITY, 0, FIXED, (23, 24, 23)), (O.ELASTICITY, 0, FIXED, (23, 24, 24)),
         (O.ELASTICITY, 1, FREE, (46, 45, 40)), (O.ELASTICITY, 1, FIXED, (35, 36, 35)), (O.ELASTICITY, 1, FIXED, (36, 36, 35)),
         (O.NS_SUPG, 1, FREE, (21, 21, 22)), (O.NS_SUPG, 1, FREE, (22, 22, 21)), (O.NS_SUPG, 1, FREE, (62, 62, 62)),
         (O.NS_SUPG, 1, FREE, (63, 62, 62)), (O.ELASTICITY, 1, FIXED, (73, 74, 74)), (O.ELASTICITY, 1, FIXED, (74, 74, 74)),
         (O.ELASTICITY, 0, FIXED, (84, 84, 85)), (O.ELASTICITY, 0, FIXED, (84, 85, 85)),
         (O.ELASTICITY, 0, FREE, (99, 100, 100)), (O.ELASTICITY, 0, FREE, (100, 100, 100)),
         (O.MASS, 1, FREE, (125, 126, 126)), (O.MASS, 1, FREE, (127, 126, 126))]


# (scalar rows are the same in both numberings, and the lines of large grids the node-major rows')
CASES = [(*c, k) for c in LINES for k in (0, 1)
         if k == 0 or (c[0] in (O.ELASTICITY, O.NS_SUPG) and np.prod(c[3]) < 100000)]


@pytest.mark.parametrize("kind,prec,fixed,n,numbering", CASES)
def test_both_sides(mf, kind, prec, fixed, n, numbering):
    print("[case] grid line", kind, prec, fixed, n, numbering, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n, jitter=0.1, seed=2)
    nf, ep, src, st = inputs(kind, mesh, prec)
    mask = (np.random.default_rng(8).random(nf * mesh.n_nodes) < 0.02).astype(np.uint8) if fixed else None
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf, numbering=numbering)
    assert pat.grid()[0]
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    assert pat.status()[0] == mf.OK
    Kr, dr = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask, scatter=1)
    # each side is within TOL of the exact rows
    assert rowscaled_gpu(pat, K, Kr) <= 2 * TOL[prec]
    assert float((d - dr).abs().max() / dr.abs().max()) <= 2 * TOL[prec]
