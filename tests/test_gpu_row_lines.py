"""Bricks on both sides of each line between scalar rows with the geometry and element blocks, and between
rows in node order and in bands of a grid's planes, against the independent scatter."""
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
GRID, RANDOM = False, True
# the last size of one way and the first of the other
LINES = [(O.MASS, 0, FIXED, GRID, (48, 49, 48)), (O.MASS, 0, FIXED, GRID, (49, 49, 48)),
         (O.MASS, 1, FIXED, GRID, (46, 46, 47)), (O.MASS, 1, FIXED, GRID, (47, 46, 47)),
         (O.POISSON, 0, FREE, RANDOM, (27, 27, 27)), (O.POISSON, 0, FREE, RANDOM, (28, 27, 27)),
         (O.MASS, 1, FREE, RANDOM, (25, 25, 25)), (O.POISSON, 1, FREE, RANDOM, (25, 26, 25)),
         (O.POISSON, 0, FIXED, RANDOM, (24, 24, 24)), (O.MASS, 0, FIXED, RANDOM, (24, 25, 24)),
         (O.POISSON, 1, FIXED, RANDOM, (20, 20, 19)), (O.POISSON, 1, FIXED, RANDOM, (20, 20, 20)),
         (O.ELASTICITY, 0, FIXED, GRID, (57, 57, 5)), (O.ELASTICITY, 0, FIXED, GRID, (58, 57, 5)),
         (O.ELASTICITY, 1, FIXED, GRID, (60, 61, 13)), (O.ELASTICITY, 1, FIXED, GRID, (62, 60, 13)),
         (O.NS_SUPG, 0, FREE, GRID, (36, 37, 2)), (O.NS_SUPG, 0, FREE, GRID, (37, 37, 2)),
         (O.NS_SUPG, 1, FIXED, GRID, (38, 38, 8)), (O.NS_SUPG, 1, FIXED, GRID, (39, 38, 8))]


@pytest.mark.parametrize("kind,prec,fixed,random,n", LINES)
def test_both_sides(mf, kind, prec, fixed, random, n):
    print("[case] row line", kind, prec, fixed, random, n, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n, jitter=0.1, seed=2)
    if random:
        mesh = W.permute_mesh(mesh, 4)[0]
    nf, ep, src, st = inputs(kind, mesh, prec)
    mask = (np.random.default_rng(8).random(nf * mesh.n_nodes) < 0.02).astype(np.uint8) if fixed else None
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf)
    assert pat.grid()[0] == (not random)
    K, d = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask)
    assert pat.status()[0] == mf.OK
    Kr, dr = assemble(mf, pat, kind, mesh, prec, ep, src, st, mask, scatter=1)
    # each side is within TOL of the exact rows
    assert rowscaled_gpu(pat, K, Kr) <= 2 * TOL[prec]
    assert float((d - dr).abs().max() / dr.abs().max()) <= 2 * TOL[prec]
