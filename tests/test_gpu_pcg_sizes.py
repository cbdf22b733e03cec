"""PCG on tridiagonal systems with as many partial sums as either width of the one-block reductions takes."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("call", ["pcg", "noalloc"])
@pytest.mark.parametrize("n", [255, 257, 32768, 32769, 131072, 131073])  # 512 and 513 partials of products, of vectors
def test_known_solution(mf, n, call):
    """b = A x for a known x; A has eigenvalues in [1, 5], so |x - x*| <= |b - A x| <= tol |b| <= 5 tol |x*|."""
    print("[case] tridiagonal", n, call, file=sys.stderr, flush=True)
    i = np.arange(n)
    cols = np.stack([i - 1, i, i + 1], 1)
    keep = (cols >= 0) & (cols < n)
    vals = np.broadcast_to(np.array([-1.0, 3.0, -1.0]), (n, 3))
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    x = np.random.default_rng(n).standard_normal(n)
    b = 3.0 * x
    b[1:] -= x[:-1]
    b[:-1] -= x[1:]
    got, tol = torch.empty(n, dtype=torch.float64, device="cuda"), 1e-10
    solve = mf.pcg if call == "pcg" else mf.pcg_noalloc
    _, res = solve(cu(rp), cu(cols[keep].astype(np.int32)), cu(vals[keep]), cu(b), got, tol=tol)
    assert res["converged"] and res["true_relres"] <= tol
    assert np.linalg.norm(got.cpu().numpy() - x) <= 5 * tol * np.linalg.norm(x) + 1e-14 * np.linalg.norm(x)
