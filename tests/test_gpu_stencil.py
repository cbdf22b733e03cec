"""Scalar multigrid levels as stencils: one cycle against the oracle at level sizes on both sides
of each coarsest-level kernel, and solves whose operator is the cycle's level 0, also after the
matrix changed, against solves on copied CSR arrays."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_multigrid import TOL, gpu_cycle, oracle_cycle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


# coarsest rows: 1000 and 1024 (one row per thread), 1089 and 3375 (one workgroup, CSR), 4913 (sweeps)
CASES = [((1, 1, 1), dict(max_levels=1)), ((9, 9, 9), dict(max_levels=1)), ((15, 7, 7), dict(max_levels=1)),
         ((10, 10, 8), dict(max_levels=1)), ((14, 14, 14), dict(max_levels=1)), ((16, 16, 16), dict(max_levels=1)),
         ((16, 16, 16), dict(max_levels=1, coarse_sweeps=0)), ((12, 8, 6), dict(coarse_rows=1)),
         ((12, 8, 6), dict(coarse_rows=1, pre_sweeps=1, post_sweeps=1)), ((4, 2, 6), dict(coarse_rows=1, coarse_sweeps=1)),
         ((8, 8, 8), dict(coarse_rows=1, pre_sweeps=0, post_sweeps=1)), ((8, 8, 8), dict(coarse_rows=1, coarse_sweeps=0))]


@pytest.mark.parametrize("dims,opts", CASES)
def test_cycle_matches_oracle(mf, dims, opts):
    say("stencil cycle", dims, opts)
    mesh = W.structured_mesh(dims, jitter=0.15, seed=3)
    mask = W.boundary_node_mask(mesh.shape) if min(dims) > 1 else None
    r = np.random.default_rng(8).standard_normal(mesh.n_nodes)
    mg, z = gpu_cycle(mf, mesh, 1, mf.Form(mf.POISSON, coef=1.3), [{"coef": 1.3}] * 8, None, mask, O.NODE_MAJOR, r, **opts)
    n_levels = len(mg.levels())
    zr = oracle_cycle(dims, mesh, 1, O.POISSON, [{"coef": 1.3}] * n_levels, n_levels, None, mask, O.NODE_MAJOR, r,
                      pre=opts.get("pre_sweeps", 2), post=opts.get("post_sweeps", 2),
                      coarse_sweeps=opts.get("coarse_sweeps", 20))
    assert np.abs(z - zr).max() <= TOL * max(np.abs(zr).max(), 1e-300)


@pytest.mark.parametrize("changed", [False, True])
@pytest.mark.parametrize("solver", ["pcg", "bicgstab"])
@pytest.mark.parametrize("dims", [(12, 8, 10), (2, 4, 2), (17, 5, 6)])
def test_solves_on_the_cycles_rows(mf, dims, solver, changed):
    say("stencil solve", dims, solver, "changed", changed)
    mesh = W.structured_mesh(dims, jitter=0.15, seed=3)
    dev = torch.device("cuda:0")
    pat = mf.Pattern(torch.from_numpy(mesh.conn).to(dev), mesh.n_nodes, 3, 1)
    coords = torch.from_numpy(mesh.coords).to(dev)
    src = torch.from_numpy(W.uniform_nodal(1, mesh.n_nodes, -1, 1, 4)).to(dev)
    mask = torch.from_numpy(W.boundary_node_mask(mesh.shape)).to(dev)
    form = mf.Form(mf.POISSON, coef=1.3)
    K, d = pat.assemble(form, coords, nodal_src=src, dirichlet=mask)
    mg = mf.Multigrid(pat, coarse_rows=8)
    mg.update(form, coords, K, dirichlet=mask)
    if changed:
        K.mul_(2.5)  # the solve is for the matrix that it is given
    rp, ci, _ = pat.arrays()
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(dev)
    solve = mf.pcg if solver == "pcg" else mf.bicgstab
    kw = dict(tol=1e-11, precond=mf.PRECOND_MG, mg=mg)
    x, res = solve(*pat.device_arrays()[:2], K, d, **kw)
    xc, resc = solve(t(rp), t(ci), K, d, **kw)
    assert res["converged"] and resc["converged"]
    import scipy.sparse as sp
    import scipy.sparse.linalg as spl
    A = sp.csr_matrix((K.cpu().numpy(), ci, rp))
    ref = spl.spsolve(A.tocsc(), d.cpu().numpy())
    # relative residual 1e-11 times the condition number of these grids (below 1e3)
    for got in (x, xc):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("pre,post", [(2, 2), (1, 0), (0, 1)])
@pytest.mark.parametrize("numbering", [0, 1])
@pytest.mark.parametrize("dims", [(4, 2, 6), (10, 8, 12)])
def test_flow_cycle_on_ragged_boxes(mf, dims, numbering, pre, post, shift):
    """Four fields, vectors at 16-byte addresses and (shift) 8 bytes past them."""
    say("flow cycle", dims, "numbering", numbering, pre, post, "shift", shift)
    import oracle.multigrid as MG
    mesh = W.structured_mesh(dims, jitter=0.15, seed=3)
    prm = [{"rho": 1.0, "mu": 0.05, "tau_m": 2e-3 * (l + 1), "tau_c": 1e-2} for l in range(8)]
    st = W.uniform_nodal(4, mesh.n_nodes, -1, 1, 5)
    mask = W.dof_mask(W.boundary_node_mask(mesh.shape), 4, field_major=bool(numbering), fields=[0, 1, 2])
    r = np.random.default_rng(8).standard_normal(4 * mesh.n_nodes)
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    pat = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, 4, numbering=numbering)
    form, coords, s, m = mf.Form(mf.NS_SUPG, **prm[0]), cuda(mesh.coords), cuda(st), cuda(mask)
    room = torch.empty(pat.nnz + 1, dtype=torch.float64, device="cuda")
    K, _ = pat.assemble(form, coords, lin_state=s, dirichlet=m, K=room[shift:shift + pat.nnz])
    mg = mf.Multigrid(pat, coarse_rows=1, pre_sweeps=pre, post_sweeps=post, tau_m=[p["tau_m"] for p in prm],
                      tau_c=[p["tau_c"] for p in prm])
    mg.update(form, coords, K, lin_state=s, dirichlet=m)
    rg, zg = (torch.zeros(r.size + 1, dtype=torch.float64, device="cuda")[shift:shift + r.size] for _ in range(2))
    rg.copy_(torch.from_numpy(r))
    z = mg.apply(rg, zg).cpu().numpy()
    n = len(mg.levels())
    levels = MG.build_levels(dims, mesh.coords, 4, O.NS_SUPG, prm[:n], n, state=st, dirichlet=mask, numbering=numbering)
    zr = MG.vcycle(levels, r, omega=0.5, pre=pre, post=post, coarse_sweeps=20)
    assert np.abs(z - zr).max() <= TOL * np.abs(zr).max()
