"""mf_mg_update reports the first level whose assembly went wrong, and is good again after a good update."""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("kind,nf", [(O.POISSON, 1), (O.ELASTICITY, 3)])
@pytest.mark.parametrize("bad", ["level1", "level2", "param"])
def test_bad_level(mf, kind, nf, bad):
    print("[case] multigrid status", kind, bad, file=sys.stderr, flush=True)
    n = (8, 8, 8)
    mesh = W.structured_mesh(n)
    pat, coords = mf.Pattern(cuda(mesh.conn), mesh.n_nodes, 3, nf), cuda(mesh.coords)
    form = mf.Form(kind, coef=1.0, nu=0.3 if nf == 3 else 0.0)
    mg = mf.Multigrid(pat, coarse_rows=1)
    assert len(mg.levels()) == 4
    ep = torch.ones(mesh.n_elems, dtype=torch.float64, device="cuda")
    K, _ = pat.assemble(form, coords, elem_param=ep)
    r = torch.ones(pat.n_rows, dtype=torch.float64, device="cuda")
    mg.update(form, coords, K, elem_param=ep)
    z = mg.apply(r).clone()
    wrong, wep = coords.clone(), ep.clone()
    if bad == "param":
        wep[5] = float("nan")
    else:  # a node of the second (and third) grid goes through its neighbours; level 0 is the caller's
        at = {"level1": 2, "level2": 4}[bad]
        wrong[:, at + 9 * (at + 9 * at)] += 3.0
    with pytest.raises(mf.MFError) as err:
        mg.update(form, wrong, K, elem_param=wep)
    assert err.value.status == (mf.ERR_NONFINITE if bad == "param" else mf.ERR_BAD_JACOBIAN)
    with pytest.raises(mf.MFError):
        mg.apply(r)
    mg.update(form, coords, K, elem_param=ep)
    assert float((mg.apply(r) - z).abs().max()) <= 1e-12 * float(z.abs().max())
