"""FP32 rows on a mesh with more than 1 GiB of element records: the sums stay in
FP64 and are rounded once."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_rows_round_once(mf):
    """The flow tangent of 636 thousand bricks in an order that is no grid's, in FP32 and in FP64.
    Both form their sums in FP64, of at most 64 products a row entry
    and element pair, so an FP32 entry is one rounding (2^-24 of it) from the FP64 one, but for the
    FP64 sums' own order: 64 * 2^-53 of the row's largest entry, here with a margin of 16."""
    n = (87, 86, 85)
    print("[case] large FP32 rows", n, file=sys.stderr, flush=True)
    mesh = W.structured_mesh(n, jitter=0.1, seed=2)
    conn = torch.from_numpy(np.ascontiguousarray(mesh.conn[:, ::-1])).cuda()
    state = torch.from_numpy(W.uniform_nodal(4, mesh.n_nodes, -1, 1, 7).astype(np.float32)).cuda()
    pat = mf.Pattern(conn, mesh.n_nodes, 3, 4)
    assert not pat.grid()[0] and mesh.n_elems * (8 * 25 * 8 + 8 * 4 * 4) > 1 << 30
    form = mf.Form(mf.NS_SUPG, rho=1.1, mu=0.02, tau_m=3e-3, tau_c=1e-2)
    coords = torch.from_numpy(mesh.coords).cuda()
    K, _ = pat.assemble(form, coords, precision=mf.F32, lin_state=state)
    K64, _ = pat.assemble(form, coords, lin_state=state.double())
    assert pat.status()[0] == mf.OK
    rp = torch.from_numpy(pat.arrays()[0]).cuda().long()
    step, over = 1 << 17, 0
    for r0 in range(0, rp.numel() - 1, step):
        r1 = min(rp.numel() - 1, r0 + step)
        k0, k1 = int(rp[r0]), int(rp[r1])
        a, b = K[k0:k1].double(), K64[k0:k1]
        row = torch.repeat_interleave(torch.arange(r1 - r0, device="cuda"), rp[r0 + 1:r1 + 1] - rp[r0:r1])
        top = torch.zeros(r1 - r0, dtype=torch.float64, device="cuda").scatter_reduce_(0, row, b.abs(), "amax")
        over += int(((a - b).abs() > 2.0 ** -24 * b.abs() + 16 * 64 * 2.0 ** -53 * top[row]).sum())
    assert over == 0
